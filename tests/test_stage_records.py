"""CPU: the record bound that a plan reports is the one its stages keep, also in whole-state programs."""
import pytest

from workloads import qft, random_layers, random_mixed_circuit

import paper_1412_2293_amd as q


@pytest.mark.parametrize("dtype,entries", [(q.C64, 1024), (q.C128, 512)], ids=["c64", "c128"])
@pytest.mark.parametrize("n", [9, 12, 14, 18])
def test_reported_stage_bound_is_eight_kib_and_kept(n, dtype, entries):
    for c in (random_layers(n, 12, n, "random"), random_mixed_circuit(n, 300, n), qft(n, n)):
        for plan in (None, {"fuse": 1}):
            d = q.plan_describe(c.gates, n, dtype, plan)
            if not d["fused"]:
                continue
            assert d["stage_rec_cap"] == entries
            for p in d["passes"]:
                assert all(s["rec_end"] - s["rec_begin"] <= entries for s in p["stages"])
