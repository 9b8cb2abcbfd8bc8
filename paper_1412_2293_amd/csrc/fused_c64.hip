// The fused pass kernels for complex<float> (one file per amplitude type, so that they compile side by
// side).
#include "fused_kernel.h"

namespace qs {

template hipError_t fused_attributes<float>();
template hipError_t fused_launch<float>(float *, int, int, const PassDesc &, int, int, int64_t, int64_t, const RunParams *,
                                      ProgramDev, const void *, const void *, const uint64_t *, size_t, hipStream_t,
                                      double *, int, int);

}  // namespace qs
