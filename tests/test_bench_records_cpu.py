"""bench.py's HBM traffic per attention launch comes from committed counter
records that are keyed to the kernel's source: an edit of the source leaves the
benchmark without them (traffic null) until they are taken again."""

import json
import os

import pytest

import bench


@pytest.mark.parametrize("workload", ["c2", "c3", "c4", "c5"])
def test_attention_traffic_records_are_of_the_current_source(workload):
    with open(os.path.join(bench.ROOT, "profiles", f"attention_{workload}_traffic.json")) as f:
        kernels = json.load(f)["by_kernel"]
    assert kernels
    for kernel in kernels:
        assert bench.kernel_traffic("k_attention.hip", workload, kernel), kernel
