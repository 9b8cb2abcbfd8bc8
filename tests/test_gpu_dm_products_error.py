"""GPU: collected products of diagonal ops against extended precision (numpy long double).

Twelve equal layers of diagonal ops whose factors are exact in FP32, between dense ops that
round nothing.  Applied one by one, every op rounds every amplitude it reaches.  A collected product
must round them once: its error may be no larger than the one-by-one form's (tiles of four registers,
which never collect).  With plain products it was larger: the error of a product is the same in every
layer, so that it grows with the layers and not with their square root."""

import numpy as np
import pytest

from workloads import DIAG, U2, Circuit, Gate

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402
from test_gpu_dm_fused import ideal_state, rho_logical  # noqa: E402

pytestmark = pytest.mark.gpu

HH = np.kron(np.array([[1, 1], [1, -1]]), np.array([[1, 1], [1, -1]])).astype(complex) / 2
FLIP0 = np.kron(np.eye(2), np.array([[0.0, 1.0], [1.0, 0.0]])).astype(complex)   # index: bit q1, then bit q0


def layers(n, seed):
    rng = np.random.default_rng(seed)
    gates = [Gate(U2, q0=t, q1=t + 1, m=HH) for t in range(0, n - 1, 2)]
    # qubit 0 with each other one, six factors each
    step = [Gate(DIAG, m=np.array([complex(rng.integers(600, 780), rng.integers(640, 820)) / 1024]),
                 mask=1 | 1 << b, value=1 | 1 << b) for _ in range(6) for b in range(2, n)]
    for _ in range(12):
        gates += step
        gates += [Gate(U2, q0=0, q1=1, m=FLIP0) for _ in range(2)]
    for i, g in enumerate(gates):
        g.site = i
    return Circuit(n, gates, name="layers", init_index=0)


def exact_state(c, dtype):
    """The pure state in long double, with the dense gates' entries as the type holds them."""
    psi = np.zeros(1 << c.n, np.clongdouble)
    psi[c.init_index] = 1
    idx = np.arange(1 << c.n)
    for g in c.gates:
        if g.kind == DIAG:
            psi[(idx & g.mask) == g.value] *= np.clongdouble(np.ravel(g.m)[0])
            continue
        m = np.asarray(g.m).reshape(4, 4).astype(np.complex64 if dtype == q.C64 else np.complex128)
        loc = (idx >> g.q0 & 1) + 2 * (idx >> g.q1 & 1)
        base = idx & ~(1 << g.q0 | 1 << g.q1)
        out = np.zeros_like(psi)
        for k in range(4):
            out += m.astype(np.clongdouble)[loc, k] * psi[base | (k & 1) << g.q0 | (k >> 1) << g.q1]
        psi = out
    return psi


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("n,tile,reg,run", [(6, 9, 4, 3), (6, 8, 3, 2), (5, 9, 4, 4)])
def test_error_no_larger_than_one_by_one(n, tile, reg, run, dtype):
    c = layers(n, 3 + n)
    psi = exact_state(c, dtype)
    want = np.outer(psi, psi.conj())
    err = []
    for plan in ({"fuse": 1, "tile_bits": tile, "reg_bits": reg, "run_bits": run},
                 {"fuse": 1, "tile_bits": tile, "reg_bits": 2, "run_bits": run}):
        d = q.plan_describe(q.dm_superop(c.gates, n, 0.0), 2 * n, dtype, plan)
        assert any(p["defer"] for p in d["passes"]) == (plan["reg_bits"] > 2)
        res = q.dm_run(c.gates, n, c.init_index, dtype, ideal_state(n, dtype, psi.astype(np.complex128)), plan=plan)
        got = rho_logical(res, n, dtype).astype(np.clongdouble)
        err.append(float(np.sqrt(np.sum(np.abs(got - want) ** 2) / np.sum(np.abs(want) ** 2))))
    assert err[0] <= err[1]
