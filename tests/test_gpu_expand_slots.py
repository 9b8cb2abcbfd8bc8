"""GPU: expanding passes whose workgroups take several slots (two and four, the last group partly filled) and
several tiles, with the overlaps formed beside them: full states of every slot, norms and fidelities against the
oracle in both dtypes.  The shape of the last pass's launch is worked out from the plan and asserted.

Tolerances as for every trajectory run: complex<double> 1e-12 relative, complex<float> 3e-5 on states and
1e-5 on fidelities."""
import numpy as np
import pytest

import oracle
from test_gpu_expand import once_per_qubit
from workloads import qft

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


def launch_shape(d, n, slots):
    """(slots per workgroup, tiles per workgroup, outer jobs) of the last pass for `slots` slots."""
    p = d["passes"][-1]
    assert p["expand"]
    walked = n - d["K"] - bin(p["classical"]).count("1")
    jobs = p["job_end"] - p["job_begin"]
    run = 2 if walked >= 12 and jobs == 0 else 1
    per = 4
    while per > 1 and ((1 << walked) // run) * -(-slots // per) < 1024:
        per //= 2
    return per, run, jobs


@pytest.mark.parametrize("make,n,seed,T,plan,per,run,jobs", [
    (qft, 19, 1, 3, (10, 3, 1), 2, 1, False),           # pairs of slots, the second half filled
    (qft, 19, 1, 7, (10, 3, 1), 4, 1, False),           # fours, the second with three
    (once_per_qubit, 20, 2, 5, (11, 3, 2), 4, 1, False),
    (once_per_qubit, 20, 3, 3, (10, 3, 1), 2, 1, True),  # with phases that depend on the tile
    (once_per_qubit, 21, 3, 5, (10, 3, 4), 4, 1, True),
    (qft, 21, 1, 6, (12, 4, 1), 4, 1, False),
    (qft, 22, 1, 5, (10, 3, 3), 4, 2, False),           # two tiles per workgroup
    (once_per_qubit, 22, 2, 6, (10, 3, 4), 4, 2, False),
])
def test_several_slots_and_tiles_per_workgroup(make, n, seed, T, plan, per, run, jobs):
    plan = {"fuse": 1, "tile_bits": plan[0], "reg_bits": plan[1], "run_bits": plan[2]}
    c, e = make(n, seed), 0.05
    want = [oracle.sv_run(c, e if s else 0.0, 17, max(s - 1, 0)) for s in range(T + 1)]
    print(f"oracle done: n={n} T={T}", flush=True)
    F_ref = np.array([abs(np.vdot(want[0], w)) ** 2 / (np.vdot(want[0], want[0]).real * np.vdot(w, w).real) for w in want[1:]])
    idx = np.arange(1 << n)
    for dtype in (q.C64, q.C128):
        d = q.plan_describe(c.gates, n, dtype, plan)
        assert launch_shape(d, n, T)[:2] == (per, run) and (launch_shape(d, n, T)[2] > 0) == jobs
        assert T % per != 0
        res = q.run_trajectories(c.gates, n, c.init_index, dtype, T, e=e, seed=17, plan=plan)
        got = q.trajectory_states(res, n, dtype, T)
        phys = np.zeros_like(idx)
        for b in range(n):
            phys |= ((idx >> b) & 1) << int(res["layout"][b])
        for slot in range(T + 1):
            g = got[slot].cpu().numpy().astype(np.complex128)
            err = np.linalg.norm(g[phys] - want[slot]) / np.linalg.norm(want[slot])
            assert err <= (1e-12 if dtype == q.C128 else 3e-5), (slot, err)
            if slot:
                assert abs(res["norm"][slot - 1] - np.sum(np.abs(g) ** 2)) <= 1e-11
        assert np.max(np.abs(res["F"] - F_ref)) <= (1e-12 if dtype == q.C128 else 1e-5)
