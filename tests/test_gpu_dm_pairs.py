"""GPU: controlled phases and CNOTs on both sides of a density matrix in one sweep, and two-qubit
Kraus sets on the matrix cores, against the dense product, for every order and kind of qubit pair at
the smallest matrices of each route (two qubits, and five for the matrix cores) and a larger one.

Tolerance: relative to the largest entry, 1e-13 in double precision (products of at most 16 terms of
operators of norm one), 1e-5 in single."""
import numpy as np
import pytest

from workloads import CNOT, CP, NOISE_PHASE, Gate

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


def dense(n, q0, q1, m):
    """The 4 x 4 operator m (local index bit(q0) + 2 bit(q1)) on n qubits."""
    N = 1 << n
    i = np.arange(N)
    loc = ((i >> q0) & 1) + 2 * ((i >> q1) & 1)
    rest = i & ~((1 << q0) | (1 << q1))
    U = np.zeros((N, N), np.complex128)
    for b in range(4):
        U[i, rest | ((b & 1) << q0) | ((b >> 1) << q1)] = m[loc, b]
    return U


def pairs(n):
    return [(a, b) for a in range(n) for b in range(n) if a != b] if n <= 5 else [(0, n - 1), (n - 1, n - 2), (1, 0), (3, 5)]


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("n", [2, 4, 5, 8])
def test_two_sided_pairs(n, dtype):
    rng = np.random.default_rng(n)
    N = 1 << n
    rho = q.StateVector(2 * n, dtype, 1)
    amps = rho.amplitudes()
    tol = 1e-13 if dtype == q.C128 else 1e-5
    for k, (a, b) in enumerate(pairs(n)):
        M = rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N))
        M = M.astype(np.complex64 if dtype == q.C64 else np.complex128)
        theta, e = float(rng.uniform(-4, 4)), 0.3
        sel = ((np.arange(N) >> a) & (np.arange(N) >> b) & 1).astype(bool)
        W = M.astype(np.complex128)
        ph = np.where(sel, np.exp(-1j * theta), 1.0)
        damp = np.where(sel[:, None] ^ sel[None, :], np.exp(-0.5 * e * e), 1.0)
        cn = np.eye(4)[[0, 3, 2, 1]]
        C = dense(n, a, b, cn)
        ops = rng.standard_normal((3, 4, 4)) + 1j * rng.standard_normal((3, 4, 4))
        ops /= np.linalg.norm(ops)
        E = [dense(n, a, b, o) for o in ops]
        cases = [
            (lambda: q.dm_apply_gate(rho, Gate(CP, q0=a, q1=b, theta=theta), 0.0), ph[:, None] * W * ph.conj()[None, :]),
            (lambda: q.dm_apply_gate(rho, Gate(CP, q0=a, q1=b, theta=theta, noise=NOISE_PHASE), e),
             ph[:, None] * W * ph.conj()[None, :] * damp),
            (lambda: q.dm_apply_gate(rho, Gate(CNOT, q0=a, q1=b), 0.0), C @ W @ C.T),
            (lambda: q.apply_kraus(rho, [a, b], ops), sum(x @ W @ x.conj().T for x in E)),
        ]
        for j, (call, want) in enumerate(cases):
            amps.copy_(torch.as_tensor(M).to(amps.device).reshape(amps.shape))
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            got = amps.cpu().numpy().astype(np.complex128).reshape(N, N)
            assert np.abs(got - want).max() <= tol * np.abs(M).max(), (a, b, j)
