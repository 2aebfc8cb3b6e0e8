"""The HBM traffic that bench.py reports from stored profiles is of the kernel that runs, or is left out."""
import json
import os

import bench
import paper_2407_20496_amd as hinm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_stored_traffic_is_of_the_kernel_that_runs():
    with open(os.path.join(ROOT, "profiles", "traffic.json")) as f:
        stored = json.load(f)
    assert len(stored) >= 14
    for key, entry in stored.items():
        c = bench.workloads()[key]
        ld = c.N if c.N == 1 else (c.N + 7) // 8 * 8
        plan = hinm.hinm_spmm_prepared_plan(c.M, c.K, c.V, c.Kv, c.dtype, c.N, ld, ld)[0]
        nbytes, source = bench.stored_traffic(key, False, plan)
        assert nbytes == entry["fetch_bytes"] + entry["write_bytes"], (key, plan)
        path = os.path.join(ROOT, source.split("run: ")[1].split(" ")[0])
        assert entry["kernel"] + "<" in open(path).read(), path
        assert bench.stored_traffic(key, False, "another_kernel<>") == (None, None)
