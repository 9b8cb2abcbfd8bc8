"""CPU: which automatic plans are whole-state programs.  Circuits whose first gates work on few tiles, or with
many dense two-qubit gates, ran slower as such programs on a full chip and stay fused passes; so do density
matrices of six and seven qubits, whose superoperators are dense.  The choice does not depend on the batch."""
import numpy as np
import pytest

from workloads import CNOT, CP, U1, U2, Circuit, Gate, grover, haar_2x2, qft, random_layers, random_mixed_circuit

import paper_1412_2293_amd as q


def whole(gates, n, dtype):
    return any(p["state"] for p in q.plan_describe(gates, n, dtype)["passes"])


@pytest.mark.parametrize("dtype,n", [(q.C64, 14), (q.C128, 13)], ids=["c64", "c128"])
def test_shallow_circuits_on_the_largest_states_run_as_passes(dtype, n):
    for c in (qft(n, 1), random_layers(n, 2, 1), random_layers(n, 5, 1), random_layers(n, 10, 1), random_layers(n, 2, 1, "random")):
        assert not whole(c.gates, n, dtype), c.name
    for c in (grover(n, 1, 1), grover(n, 1, 5), random_layers(n, 60, 1), random_layers(n, 20, 1, "random")):
        assert whole(c.gates, n, dtype), c.name


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
def test_smaller_states_run_whole(dtype):
    for n in (2, 5, 8, 10, 12):
        for c in (random_layers(n, 2, 1), random_layers(n, 20, 1, "random")):
            assert whole(c.gates, n, dtype), (c.name, n)


@pytest.mark.parametrize("dtype,first", [(q.C64, 10), (q.C128, 11)], ids=["c64", "c128"])
def test_dense_gates(dtype, first):
    for n in (first, 12, 13):
        assert not whole(random_mixed_circuit(n, 300, 5).gates, n, dtype)
    n = first - 1
    assert whole(random_mixed_circuit(n, 300, 5).gates, n, dtype)
    # the line: one dense gate in eight
    rng, n = np.random.default_rng(1), first
    for dense, expect in ((8, True), (9, False)):
        gates = [Gate(U1, q0=k % n, m=haar_2x2(rng)) for k in range(64 - dense)]
        gates[1:1] = [Gate(CNOT, q0=k % n, q1=(k + 1) % n) for k in range(dense)]
        gates += [Gate(CP, q0=0, q1=1, theta=1.0)]
        assert whole(Circuit(n, gates).gates, n, dtype) == expect


@pytest.mark.parametrize("dtype", [q.C64, q.C128], ids=["c64", "c128"])
@pytest.mark.parametrize("n", [6, 7])
def test_density_matrices_use_more_than_one_workgroup(n, dtype):
    for c in (random_layers(n, 6, 1, "random"), grover(n, 1, 3)):
        assert not whole(q.dm_superop(c.gates, n, 0.02), 2 * n, dtype)
