"""GPU: circuits whose state one workgroup holds (whole-state programs), and passes of plain
reflections that run sheared, against the oracle: the smallest and largest states of each register
tile, one and two LDS buffers, controlled phases on every thread-id bit, two-qubit and diagonal ops,
rotation noise far beyond a right angle (the factors left out get small, or change sign), replays.

Tolerances as for every trajectory run: complex<double> 1e-12 relative, complex<float> 3e-5 on
states and 1e-5 on fidelities."""
import math

import numpy as np
import pytest

import oracle
from workloads import FLIP, NOISE_ROT, U1, Circuit, Gate, grover, qft, random_layers, random_mixed_circuit

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


def check(c, dtype, plan, T, e, seed=11):
    res = q.run_trajectories(c.gates, c.n, c.init_index, dtype, T, e=e, seed=seed, plan=plan)
    F_ref, _, ideal, states = oracle.run_trajectories(c, e, seed, range(T), keep_states=True)
    got = q.trajectory_states(res, c.n, dtype, T).cpu().numpy().astype(np.complex128)
    idx = np.arange(1 << c.n)
    phys = np.zeros_like(idx)
    for b in range(c.n):
        phys |= ((idx >> b) & 1) << int(res["layout"][b])
    for slot in range(T + 1):
        want = states[slot - 1] if slot else ideal
        err = np.linalg.norm(got[slot][phys] - want) / np.linalg.norm(want)
        assert err <= (1e-12 if dtype == q.C128 else 3e-5), (c.name, slot, err)
    assert np.max(np.abs(res["F"] - F_ref)) <= (1e-12 if dtype == q.C128 else 1e-5), c.name


def tile(n, rb):
    return {"fuse": 1, "tile_bits": n, "reg_bits": rb, "run_bits": 4}


@pytest.mark.parametrize("dtype,n,plan", [
    (q.C64, 2, None), (q.C128, 3, None), (q.C64, 5, tile(5, 2)), (q.C128, 6, tile(6, 3)), (q.C64, 6, tile(6, 4)),
    (q.C128, 8, tile(8, 4)), (q.C64, 11, tile(11, 2)), (q.C128, 11, None), (q.C64, 12, tile(12, 3)),
    (q.C128, 12, tile(12, 4)), (q.C64, 12, tile(12, 4)), (q.C128, 12, None), (q.C64, 13, None), (q.C128, 13, None),
    (q.C64, 14, None),
])
def test_whole_state_programs(dtype, n, plan):
    programs = 0
    cs = [random_mixed_circuit(n, 70, 40 + n), random_layers(n, 6, n), qft(n, n)]
    if n >= 3:
        cs.append(grover(n, n, iterations=2))
    for c in cs:
        d = q.plan_describe(c.gates, n, dtype, plan) if plan else q.plan_describe(c.gates, n, dtype)
        programs += sum(p["state"] > 0 for p in d.get("passes", []))
        check(c, dtype, plan, 3, 0.1)
    assert programs > 0


@pytest.mark.parametrize("dtype,n", [(q.C64, 14), (q.C128, 13), (q.C64, 4)])
def test_whole_state_replays(dtype, n):
    c = random_mixed_circuit(n, 60, 3)
    with q.TrajGraph(c.gates, n, dtype, 4) as g:
        for k, init in enumerate((0, (1 << n) - 1, 5, 0)):
            got = g.launch(init, e=0.05, seed=k // 3)
            ref = q.run_trajectories(c.gates, n, init, dtype, 4, e=0.05, seed=k // 3)
            assert np.array_equal(got["F"], ref["F"]) and np.array_equal(got["norm"], ref["norm"])


def reflections(n, layers, seed, kind):
    """Layers of one real gate on every qubit with sign flips of one state between them.  kind: "h" Hadamards; "axis" reflections about random
    axes nearer to z than to x; "mixed" every third a rotation, which runs unsheared."""
    rng = np.random.default_rng(seed)
    gates = []
    for layer in range(layers):
        for t in range(n):
            a = math.pi / 4 if kind == "h" else rng.uniform(-math.pi / 4, math.pi / 4)
            s = -1.0 if kind != "mixed" or rng.random() < 0.7 else 1.0
            m = np.array([[math.cos(a), math.sin(a)], [-s * math.sin(a), s * math.cos(a)]], np.complex128)
            gates.append(Gate(U1, q0=t, m=m, noise=NOISE_ROT))
        gates.append(Gate(FLIP, mask=(1 << n) - 1, value=int(rng.integers(0, 1 << n))))
    for i, g in enumerate(gates):
        g.site = i
    return Circuit(n, gates, name=kind)


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("kind,e", [("h", 0.1), ("h", 40.0), ("axis", 0.3), ("axis", 40.0), ("mixed", 0.3)])
@pytest.mark.parametrize("n,plan", [(13, {"fuse": 1, "tile_bits": 12, "reg_bits": 4, "run_bits": 4}),
                                    (11, {"fuse": 1, "tile_bits": 7, "reg_bits": 3, "run_bits": 2}),
                                    (9, {"fuse": 1, "tile_bits": 5, "reg_bits": 4, "run_bits": 1})])
def test_plain_reflection_passes(n, plan, kind, e, dtype):
    c = reflections(n, 8, 5, kind)
    sheared = sum(p["shear"] for p in q.plan_describe(c.gates, n, dtype, plan)["passes"])
    assert sheared > 0 or kind == "mixed"
    check(c, dtype, plan, 4, e)


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
def test_sheared_factors_of_zero(dtype):
    """All gates share one draw, and e turns every Hadamard of trajectory 0 into X or -X (up to
    rounding): the first diagonal entry, which the sheared form leaves out, vanishes."""
    n, seed = 11, 5
    c = reflections(n, 6, 1, "h")
    for g in c.gates:
        g.site = 0
    xi = float(oracle.normals(seed, [0], [0])[0, 0])
    e = (math.pi / 4 if xi > 0 else 3 * math.pi / 4) / abs(xi)
    plan = {"fuse": 1, "tile_bits": 7, "reg_bits": 4, "run_bits": 2}
    assert any(p["shear"] for p in q.plan_describe(c.gates, n, dtype, plan)["passes"])
    check(c, dtype, plan, 2, e, seed)
