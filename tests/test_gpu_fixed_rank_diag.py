"""Fixed-rank two-qubit steps of diagonal Kraus sets (the compact Gram and recombination) against the
numpy oracle, and against the general kernels on the same set.  Sizes: one block of plain loops
(n = 5), the smallest matrix-core step (8, one 16-row step per wave), several blocks (13, 16, 19), low,
middle and high pairs in both orders, rank bounds 3 and 8.  complex<double> entries of rho within
1e-12, complex<float> fidelities within 1e-5."""
import math

import numpy as np
import pytest

from oracle import fixed_rank
from workloads import U1, Gate

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


def _haar(rng, d):
    u, r = np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    return u * (np.diag(r) / np.abs(np.diag(r)))[None, :]


def _diagonal_set(rng, n_ops):
    """A complete set of diagonal operators: columns of unit vectors on the diagonal."""
    z = rng.standard_normal((n_ops, 4)) + 1j * rng.standard_normal((n_ops, 4))
    z /= np.linalg.norm(z, axis=0)
    return np.stack([np.diag(v) for v in z])


@pytest.mark.parametrize("dtype", [q.C128, q.C64], ids=["c128", "c64"])
@pytest.mark.parametrize("n,r", [(5, 8), (8, 8), (9, 3), (13, 8)])
def test_diagonal_two_qubit_steps_against_oracle(n, r, dtype):
    rng = np.random.default_rng(40 + n)
    fr = q.FixedRank(n, r, dtype)
    ref = fixed_rank.FixedRank(n, r, init_index=1, tau=1e-9, zero_tol=1e-13)
    fr.init_basis(1)
    for k, (a, b) in enumerate([(0, 1), (n - 1, 0), (2, n - 2), (n - 2, n - 1), (3, 1)]):
        for qb in range(n):
            U = _haar(rng, 2)
            fr.apply_gate(Gate(U1, q0=qb, m=U))
            ref.apply_unitary([qb], U)
        ops = _diagonal_set(rng, 2 + k % 3)
        rank = fr.apply_kraus2(a, b, ops, zero_tol=1e-13 if dtype == q.C128 else 1e-6)
        ref.apply_kraus([a, b], ops)
        if dtype == q.C128:
            assert rank == len(ref.V)
    rank, lt = fr.info()
    V = fr.columns()[:rank].cpu().numpy().astype(np.complex128).T
    if dtype == q.C128:
        np.testing.assert_allclose(math.exp(lt) * (V @ V.conj().T), ref.rho(), atol=1e-12)
    psi = np.exp(1j * rng.uniform(0, 2 * np.pi, 1 << n)) / math.sqrt(1 << n)
    fn = float(np.sum(np.abs(psi.conj() @ V) ** 2))
    fu_ref, fn_ref, lt_ref = ref.fidelity(psi)
    tol = 1e-11 if dtype == q.C128 else 1e-5
    assert abs(fn - fn_ref) <= tol and abs(fn * math.exp(lt) - fu_ref) <= tol and abs(lt - lt_ref) <= tol


@pytest.mark.parametrize("n", [16, 19])
def test_diagonal_step_equals_the_general_form(n):
    """The same set with an off-diagonal entry of 1e-300 takes the general kernels."""
    rng = np.random.default_rng(n)
    ops = _diagonal_set(rng, 2)
    near = ops.copy()
    near[0, 0, 1] = 1e-300
    out = []
    for o in (ops, near):
        g = np.random.default_rng(3)
        fr = q.FixedRank(n, 8, q.C128)
        fr.init_basis(0)
        for k, (a, b) in enumerate([(0, n - 1), (5, 4), (n - 3, 2), (1, 9), (7, n - 2)]):
            for qb in (a, b):
                fr.apply_gate(Gate(U1, q0=qb, m=_haar(g, 2)))
            fr.apply_kraus2(a, b, o)
        rank, lt = fr.info()
        out.append((rank, lt, fr.columns()[:rank].clone()))
    assert out[0][0] == out[1][0] and abs(out[0][1] - out[1][1]) <= 1e-12
    a, b = out[0][2], out[1][2]
    G = (a.conj() @ b.T).cpu().numpy()     # equal up to a phase per column
    assert np.allclose(np.sum(np.abs(G) ** 2), np.sum(np.abs((a.conj() @ a.T).cpu().numpy()) ** 2), atol=1e-11)


@pytest.mark.parametrize("n", [16, 19])
def test_diagonal_steps_give_the_general_density_matrix(n):
    """||rho_a - rho_b||_F of the compact and the general form, so that components outside the other's columns
    count too: with the columns side by side, M = (A, B) = Q R, it is the norm of R diag(1, -1) R^dagger.  Both
    round each of five steps to about 1e-15 of their Gram matrices and truncate to the same rank, an error that
    grows by the inverse gap of the spectrum there; 1e-10 leaves a factor of 10^4 for it."""
    rng = np.random.default_rng(100 + n)
    ops = _diagonal_set(rng, 3)
    near = ops.copy()
    near[0, 0, 1] = 1e-300
    cols, ranks = [], []
    for o in (ops, near):
        g = np.random.default_rng(4)
        fr = q.FixedRank(n, 8, q.C128)
        fr.init_basis(1)
        for k, (a, b) in enumerate([(0, n - 1), (n - 2, 1), (3, 2), (n - 4, 8), (6, n - 1)]):
            for qb in (a, b):
                fr.apply_gate(Gate(U1, q0=qb, m=_haar(g, 2)))
            ranks.append(fr.apply_kraus2(a, b, o))
        rank, lt = fr.info()
        cols.append(fr.columns()[:rank].cpu().numpy().T * math.exp(0.5 * lt))
    assert ranks[:5] == ranks[5:] and max(ranks) == 8
    r = cols[0].shape[1]
    R = np.linalg.qr(np.hstack(cols), mode="r")
    dist = np.linalg.norm(R @ np.diag([1.0] * r + [-1.0] * r) @ R.conj().T)
    assert dist <= 1e-10, dist
