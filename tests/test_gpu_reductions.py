"""GPU: the FP64 reductions at the sizes where their split changes (one step of the workgroup, a few
in flight, one block and many, rows shorter and longer than a step) against numpy in extended sums.

Tolerance: the inputs are exact in FP64, so only the rounding of sums of at most 2^22 products is
left; 1e-12 of the sum of their magnitudes covers any order of summation."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


def random_states(rng, shape, dtype):
    z = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    return z.astype(np.complex64 if dtype == q.C64 else np.complex128)


def put(sv, states):
    amps = sv.amplitudes()
    amps.copy_(torch.as_tensor(states).to(amps.device).reshape(amps.shape))
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("n,T", [(1, 1), (7, 2), (8, 1), (9, 3), (10, 1), (11, 2), (18, 1), (20, 3), (21, 1), (22, 1)])
def test_fidelity_sizes(n, T, dtype):
    rng = np.random.default_rng(n)
    a, b = q.StateVector(n, dtype, T), q.StateVector(n, dtype, T)
    A, B = random_states(rng, (T, 1 << n), dtype), random_states(rng, (T, 1 << n), dtype)
    put(a, A)
    put(b, B)
    x, y = A[T - 1].astype(np.complex128), B[0].astype(np.complex128)
    f, ov = q.fidelity(a, T - 1, b, 0)
    want = np.vdot(x, y)
    na, nb = np.vdot(x, x).real, np.vdot(y, y).real
    assert abs(ov - want) <= 1e-12 * math.sqrt(na * nb)
    assert abs(f - abs(want) ** 2 / (na * nb)) <= 1e-11


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("n", [1, 5, 7, 8, 9, 10, 11])
def test_dm_fidelity_sizes(n, dtype):
    rng = np.random.default_rng(n)
    rho, psi = q.StateVector(2 * n, dtype, 1), q.StateVector(n, dtype, 2)
    M, P = random_states(rng, (1 << n, 1 << n), dtype), random_states(rng, (2, 1 << n), dtype)
    put(rho, M)
    put(psi, P)
    M, v = M.astype(np.complex128), P[1].astype(np.complex128)
    f, tr = q.dm_fidelity(rho, psi, 1)
    scale = float(np.abs(v) @ np.abs(M) @ np.abs(v))
    assert abs(f - np.vdot(v, M @ v).real) <= 1e-12 * scale
    assert abs(tr - np.trace(M).real) <= 1e-12 * float(np.abs(np.diag(M)).sum())
