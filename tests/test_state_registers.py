"""CPU: the whole-state kernels keep their tiles in registers (the compiler's resource remarks report no scratch
memory), and complex<double> tiles of 8 amplitudes leave two workgroups of 512 threads per CU their registers."""
import os
import re
import subprocess

from paper_1412_2293_amd import build


def test_whole_state_kernels_do_not_spill(tmp_path):
    r = subprocess.run([build.hipcc(), "-x", "hip", *build.common_flags(), "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, "state.hip"), "-o", str(tmp_path / "state.o")],
                       stderr=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = re.findall(r"Function Name: (\S+).*?TotalSGPRs.*?VGPRs: (\d+).*?ScratchSize \[bytes/lane\]: (\d+)", r.stderr, re.S)
    assert len(kernels) == 12
    for name, vgprs, scratch in kernels:
        assert int(scratch) == 0, name
        if "k_stateIdLi3" in name:
            assert int(vgprs) <= 128, name
