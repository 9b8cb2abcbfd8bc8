"""Whole-state programs of deep circuits on more than 12 qubits run their slots in groups that share one record area: the run buffer
does not grow with the records of every slot (CPU), and results are the same bits in and across groups, also in
a captured graph that is replayed (GPU)."""
import numpy as np
import pytest

import oracle
from workloads import random_layers

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
def test_buffer_grows_by_states_and_noise_only(dtype):
    n = 13
    c = random_layers(n, 200, 1, "random")
    assert q.plan_describe(c.gates, n, dtype)["passes"][0]["state"]
    a, b = (q.traj_bytes_required(c.gates, n, dtype, T) for T in (10000, 20000))
    amp = 8 if dtype == q.C64 else 16
    # a slot's state, its noise-table rows, and its strength, phase products and sums
    slot = (amp << n) + len(c.gates) * 64 + 8 + amp + 5 * 8
    partials = 3 * 8 * (1 << n) // 2048
    assert (b - a) / 10000 <= slot + partials + 1


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,n", [(q.C64, 13), (q.C128, 13)])
def test_groups_do_not_change_results(dtype, n):
    T, e, seed = 1100, 0.05, 3
    c = random_layers(n, 60, 1, "random")
    d = q.plan_describe(c.gates, n, dtype)["passes"][0]
    assert d["state"] and d["rec_size"] * (8 if dtype == q.C64 else 16) * 513 > 64 << 20   # groups of 512 slots
    res = q.run_trajectories(c.gates, n, c.init_index, dtype, T, e=e, seed=seed)
    st = q.trajectory_states(res, n, dtype, T).cpu().numpy()
    for base in (0, 509, 1021, T - 3):    # the first slots, over both borders, the last
        part = q.run_trajectories(c.gates, n, c.init_index, dtype, 3, e=e, seed=seed, traj_base=base)
        for k in ("F", "norm"):
            assert np.array_equal(part[k], res[k][base:base + 3]), (base, k)
        assert np.array_equal(q.trajectory_states(part, n, dtype, 3)[1:].cpu().numpy(), st[base + 1:base + 4]), base
    F_ref, _ = oracle.run_trajectories(c, e, seed, [0, 511, 512, T - 1])
    assert np.max(np.abs(res["F"][[0, 511, 512, T - 1]] - F_ref)) <= (1e-12 if dtype == q.C128 else 3e-5)
    with q.TrajGraph(c.gates, n, dtype, T) as g:
        for s in (seed, 5, seed):
            got = g.launch(c.init_index, e=e, seed=s)
            ref = q.run_trajectories(c.gates, n, c.init_index, dtype, T, e=e, seed=s)
            assert np.array_equal(got["F"], ref["F"]) and np.array_equal(got["norm"], ref["norm"])
