"""CPU: what bench.py records."""
import json
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1412_2293_amd", "csrc")


def test_profile_key_covers_every_file_of_the_profiled_kernels():
    """The stored counters count as those of the current build only while every file that the fused passes'
    kernels are compiled from is unchanged, headers included."""
    seen, todo = set(), ["fused.hip", "fused_c64.hip", "expand.hip"]
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        text = open(os.path.join(CSRC, f)).read()
        todo += [g for g in re.findall(r'#include "([^"]+)"', text) if os.path.exists(os.path.join(CSRC, g))]
    assert seen <= set(bench.PROFILED_SOURCES)


def test_headline_line_is_short_and_whole():
    """The headline line stands alone (a record that keeps only the end of the output still parses it), and each
    side measurement has a line of its own."""
    keys = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config", "roofline")
    out = {k: {"x": 1.0} for k in keys}
    out["serving"] = {"latency_p50_s": 0.1, "latency_p99_s": 0.2, "requests": [{"n": 20}] * 500}
    out["cpu_baseline"] = {"value": 5e9, "all": list(range(2000))}
    out["sweeps_n28"] = {"q": list(range(5000))}
    details, line = bench.record(out)
    head = json.loads(line)
    assert len(line) < 4096 and "\n" not in line
    assert set(keys) <= set(head)
    assert head["serving_latency_p50_s"] == 0.1 and head["serving_latency_p99_s"] == 0.2
    assert not set(head) & set(bench.SIDE)
    side = {}
    for d in details:
        side.update(json.loads(d[len("[bench] "):]))
    assert side == {k: out[k] for k in ("serving", "cpu_baseline", "sweeps_n28")}


def test_every_side_measurement_is_named_as_such():
    """What main() adds to its result below the headline goes to the side lines."""
    src = open(os.path.join(bench.ROOT, "bench.py")).read()
    added = set(re.findall(r'^        +out\["(\w+)"\] = (?!round)', src[src.index("if not a.no_extras:"):src.index("def record")], re.M))
    assert added and added <= set(bench.SIDE)
