"""GPU: whole-state programs exchange through two LDS buffers when every slot runs at once and through one
when there are more slots: a trajectory's results are the same bits in a small and a large batch, and agree
with the oracle.  Sizes: one to six workgroups per CU with two buffers, and a tile that has room for one only.

Tolerance against the oracle as for every trajectory run: complex<double> 1e-12, complex<float> 1e-5."""
import numpy as np
import pytest

import oracle
from workloads import grover, random_layers

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,many", [(q.C64, 8, 2900), (q.C64, 10, 1600), (q.C64, 13, 300), (q.C64, 14, 300),
                                          (q.C128, 10, 800), (q.C128, 12, 300), (q.C128, 13, 300)])
def test_results_do_not_depend_on_the_number_of_slots(dtype, n, many):
    few, e, seed = 3, 0.05, 7
    for c in (random_layers(n, 5, 2, "random"), grover(n, 3, iterations=1)):
        plan = {"fuse": 1, "tile_bits": n, "reg_bits": {8: 2, 10: 2, 12: 3}.get(n, 4), "run_bits": 4}
        assert [p["state"] > 0 for p in q.plan_describe(c.gates, n, dtype, plan)["passes"]] == [True]
        res = [q.run_trajectories(c.gates, n, c.init_index, dtype, T, e=e, seed=seed, plan=plan) for T in (few, many)]
        st = [q.trajectory_states(r, n, dtype, T)[:few + 1].cpu().numpy() for r, T in zip(res, (few, many))]
        assert np.array_equal(st[0], st[1])
        for k in ("F", "norm"):
            assert np.array_equal(res[0][k], res[1][k][:few])
        F_ref, _ = oracle.run_trajectories(c, e, seed, range(few))
        assert np.max(np.abs(res[1]["F"][:few] - F_ref)) <= (1e-12 if dtype == q.C128 else 1e-5)
