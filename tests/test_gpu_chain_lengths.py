"""GPU: phase chains whose lengths lie at the edges of the lane groups that factor them (8, 16, 32, 64 and
more than one round of 64), long and short chains in one circuit: every amplitude against the oracle.

Tolerance: complex<double> 1e-12 relative, as for every trajectory run."""
import numpy as np
import pytest

import oracle
from workloads import Circuit, random_layers

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("plan", [None, {"fuse": 1, "tile_bits": 5, "reg_bits": 2, "run_bits": 2}], ids=["auto", "t5r2"])
@pytest.mark.parametrize("length", [2, 8, 9, 16, 17, 32, 33, 64, 65, 130])
def test_chain_lengths(length, plan):
    n, T, e, seed = 8, 5, 0.1, 3
    long, short = random_layers(n, length, 1, "random"), random_layers(n, 2, 2)
    # the upper half of the qubits takes only two layers, so their chains are short
    gates = [g for g in long.gates if g.q0 < n // 2 and g.q1 < n // 2] + [g for g in short.gates if g.q0 >= n // 2]
    for i, g in enumerate(gates):
        g.site = i
    c = Circuit(n, gates, name="lengths", init_index=5)
    chains = q.plan_describe(c.gates, n, q.C128, plan)["chains"]
    assert max(len(ch) for ch in chains) == length
    res = q.run_trajectories(c.gates, n, c.init_index, q.C128, T, e=e, seed=seed, plan=plan)
    F_ref, _, ideal, states = oracle.run_trajectories(c, e, seed, range(T), keep_states=True)
    got = q.trajectory_states(res, n, q.C128, T).cpu().numpy()
    idx = np.arange(1 << n)
    phys = np.zeros_like(idx)
    for b in range(n):
        phys |= ((idx >> b) & 1) << int(res["layout"][b])
    for slot in range(T + 1):
        want = states[slot - 1] if slot else ideal
        assert np.linalg.norm(got[slot][phys] - want) <= 1e-12 * np.linalg.norm(want), slot
    assert np.max(np.abs(res["F"] - F_ref)) <= 1e-12
