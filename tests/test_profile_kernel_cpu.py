"""Counters are reported for the kernel they were taken on: the names that the
profiler records carry the form of the single-query kernel (with solo runs or
without), which a name without it never matched."""
import json
import os

import pytest

from paper_1607_05707_amd import profiling

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name,block,op,same", [
    ("persistent_kernel<512, irgl::SsspOp, false>", 512, "SsspOp", True),
    ("persistent_kernel<512, irgl::SsspOp, true>", 512, "SsspOp", True),
    ("persistent_kernel<1024, irgl::BfsOp, false>", 1024, "BfsOp", True),
    ("persistent_kernel<1024, irgl::BfsOp, false>", 512, "BfsOp", False),
    ("persistent_kernel<1024, irgl::BfsOp, false>", 1024, "SsspOp", False),
    ("persistent_kernel<512, irgl::SsspOp>", 512, "SsspOp", False),  # a kernel of before
])
def test_names(name, block, op, same):
    assert profiling.is_query_kernel(name, block, op) == same


@pytest.mark.parametrize("kind,block,op", [("bfs", 1024, "BfsOp"), ("sssp", 512, "SsspOp")])
def test_committed_counters_name_a_kernel_of_the_library(kind, block, op):
    with open(os.path.join(ROOT, "profiles", f"traffic_rmat22_{kind}.json")) as f:
        assert profiling.is_query_kernel(json.load(f)["kernel"], block, op)
