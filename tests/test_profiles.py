"""The committed counter summaries (profiles/*_traffic.json) describe the kernels of this tree: the
benchmark reports a kernel's HBM traffic only while the hash of its sources is the one the counters were
taken on, so an edit to a source without a new profile takes the figure out of the report."""
import glob
import json
import os

import pytest

import bench

SUMMARIES = sorted(glob.glob(os.path.join(bench.ROOT, "profiles", "*_traffic.json")))


@pytest.mark.parametrize("path", SUMMARIES, ids=[os.path.basename(p) for p in SUMMARIES])
def test_counters_belong_to_the_present_source(path):
    with open(path) as f:
        t = json.load(f)
    name = os.path.basename(path)[:-len("_traffic.json")]
    kernel = next(k for k in bench.KERNEL_SOURCES if name.startswith(k + "_"))
    assert t["kernel_source_hash"] == bench.source_hash(bench.KERNEL_SOURCES[kernel])
    assert bench.load_traffic(kernel, name[len(kernel) + 1:]) == t["bytes_per_launch"]
