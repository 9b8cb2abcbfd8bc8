"""GPU: density-matrix passes that collect the products of their diagonal ops (tiles of 8 and 16 registers): noisy
controlled phases on every pair of qubits between gates that end a collection, patterns on one, two
(of changing pairs) and more register bits, with clear condition bits among them, against the oracle.

Tolerances as for every density-matrix run: complex<double> 1e-12 relative, complex<float> 2e-5."""

import numpy as np
import pytest

import oracle
from workloads import CP, DIAG, NOISE_PHASE, NOISE_ROT, U1, Circuit, Gate, haar_2x2, qft

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402
from test_gpu_dm_fused import ideal_state, rel_err, rho_logical  # noqa: E402

pytestmark = pytest.mark.gpu


def phases_between(n, seed):
    rng = np.random.default_rng(seed)
    gates = [Gate(U1, q0=t, m=haar_2x2(rng), noise=NOISE_ROT) for t in range(n)]
    for _ in range(3):
        for k in range(30):
            a, b = (int(x) for x in rng.choice(n, 2, replace=False))
            gates.append(Gate(CP, q0=a, q1=b, theta=float(rng.uniform(0, 6)), noise=NOISE_PHASE))
            if k % 10 == 0:
                mask = int(rng.integers(1, 1 << n))
                gates.append(Gate(DIAG, m=np.array([np.exp(1j * k)]), mask=mask, value=int(rng.integers(0, 1 << n)) & mask))
        gates.append(Gate(U1, q0=int(rng.integers(0, n)), m=haar_2x2(rng), noise=NOISE_ROT))
    for i, g in enumerate(gates):
        g.site = i
    return Circuit(n, gates, name="phases", init_index=int(rng.integers(0, 1 << n)))


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("make,n,plan", [
    (phases_between, 5, {"fuse": 1, "tile_bits": 8, "reg_bits": 4, "run_bits": 2}),
    (phases_between, 6, {"fuse": 1, "tile_bits": 9, "reg_bits": 4, "run_bits": 3}),
    (phases_between, 7, {"fuse": 1, "tile_bits": 12, "reg_bits": 4, "run_bits": 4}),
    (phases_between, 6, {"fuse": 1, "tile_bits": 8, "reg_bits": 3, "run_bits": 2}),
    (phases_between, 7, {"fuse": 1, "tile_bits": 11, "reg_bits": 3, "run_bits": 3}),
    (lambda n, s: qft(n, seed=s, x=45), 7, {"fuse": 1, "tile_bits": 12, "reg_bits": 4, "run_bits": 4}),
    (lambda n, s: qft(n, seed=s, x=9), 6, {"fuse": 1, "tile_bits": 7, "reg_bits": 4, "run_bits": 2}),
])
def test_collected_products(make, n, plan, dtype):
    c, e = make(n, 11 + n), 0.12
    d = q.plan_describe(q.dm_superop(c.gates, n, e), 2 * n, dtype, plan)
    assert any(p["defer"] for p in d["passes"])
    psi = oracle.sv_run(c, 0.0, 0, 0)
    want = oracle.dm_run(c, e)
    res = q.dm_run(c.gates, n, c.init_index, dtype, ideal_state(n, dtype, psi), e=e, plan=plan)
    assert rel_err(rho_logical(res, n, dtype), want) <= (1e-12 if dtype == q.C128 else 2e-5)
    assert abs(res["F"] - np.vdot(psi, want @ psi).real) <= (1e-12 if dtype == q.C128 else 1e-5)
