"""Passes that run as expansions (every op a real update of an untouched target with at most one
uniform output phase): full states, norms and fidelities against the oracle at the smallest and
largest tiles, with targets, touched bits and classical bits in every part of the tile, one
workgroup per slot and several slots per workgroup.

Tolerances as for every trajectory run: complex<double> 1e-12 relative, complex<float> 3e-5 on
states and 1e-5 on fidelities."""
import math

import numpy as np
import pytest

import oracle
from workloads import CP, NOISE_PHASE, NOISE_ROT, U1, Circuit, Gate, qft

torch = pytest.importorskip("torch")
import paper_1412_2293_amd as q  # noqa: E402

pytestmark = pytest.mark.gpu


def once_per_qubit(n: int, seed: int) -> Circuit:
    """Real one-qubit gates on most qubits, once each in random order, controlled phases on
    qubits not yet touched between them, from a random basis state; the rest stay classical."""
    rng = np.random.default_rng(seed)
    gates, order = [], rng.permutation(n)
    targets = order[: n - int(rng.integers(0, 3))]
    for k, t in enumerate(targets):
        a = rng.uniform(0, 2 * math.pi)
        m = np.array([[math.cos(a), math.sin(a)], [math.sin(a), -math.cos(a)]], np.complex128)
        gates.append(Gate(U1, q0=int(t), m=m, noise=NOISE_ROT))
        for c in order[k + 1:]:
            if rng.random() < 0.4:
                gates.append(Gate(CP, q0=int(c), q1=int(t), theta=float(rng.uniform(0, 6)), noise=NOISE_PHASE))
    for i, g in enumerate(gates):
        g.site = i
    return Circuit(n, gates, name="once", init_index=int(rng.integers(0, 1 << n)))


@pytest.mark.parametrize("dtype", [q.C128, q.C64], ids=["c128", "c64"])
@pytest.mark.parametrize("make,n,T,plan", [
    (qft, 10, 3, {"fuse": 1}), (qft, 11, 9, {"fuse": 1}), (qft, 12, 1, {"fuse": 1}), (qft, 18, 5, {"fuse": 1}),
    (qft, 14, 6, {"fuse": 1, "tile_bits": 10, "reg_bits": 3, "run_bits": 3}),
    (once_per_qubit, 12, 4, {"fuse": 1}), (once_per_qubit, 16, 7, {"fuse": 1}), (once_per_qubit, 17, 2, {"fuse": 1}),
    (once_per_qubit, 19, 9, {"fuse": 1}),
    (once_per_qubit, 15, 5, {"fuse": 1, "tile_bits": 11, "reg_bits": 3, "run_bits": 2}),
])
def test_expanding_passes_against_oracle(make, n, T, plan, dtype):
    e, seed = 0.05, 17
    expanded = 0
    for s in (1, 2):
        c = make(n, s)
        expanded += sum(p["expand"] for p in q.plan_describe(c.gates, n, dtype, plan)["passes"])
        res = q.run_trajectories(c.gates, n, c.init_index, dtype, T, e=e, seed=seed, plan=plan)
        got = q.trajectory_states(res, n, dtype, T).cpu().numpy().astype(np.complex128)
        idx = np.arange(1 << n)
        phys = np.zeros_like(idx)
        for b in range(n):
            phys |= ((idx >> b) & 1) << int(res["layout"][b])
        F_ref, _ = oracle.run_trajectories(c, e, seed, range(T))
        for slot in (0, 1, T):
            want = oracle.sv_run(c, e if slot else 0.0, seed, slot - 1 if slot else 0)
            err = np.linalg.norm(got[slot][phys] - want) / np.linalg.norm(want)
            assert err <= (1e-12 if dtype == q.C128 else 3e-5), (s, slot, err)
        tol = 1e-12 if dtype == q.C128 else 1e-5
        assert np.max(np.abs(res["F"] - F_ref)) <= tol
        assert np.max(np.abs(res["norm"] - np.sum(np.abs(got[1:]) ** 2, axis=1))) <= 1e-12 * 8
    assert expanded > 0
