"""The traffic counters of a stage hold for the sources they were taken on (CPU only)."""

import os
import re

import pytest

import bench


def _included(name, seen):
    text = open(os.path.join(bench.CSRC, name)).read()
    for inc in re.findall(r'^#include "([^"]+)"', text, re.M):
        if inc not in seen and os.path.exists(os.path.join(bench.CSRC, inc)):
            seen.add(inc)
            _included(inc, seen)
    return seen


@pytest.mark.parametrize("stage", list(bench.STAGE_SOURCE))
def test_hash_covers_every_source_of_the_stage(stage):
    files = set(bench.source_files(stage))
    used = {f for f in list(files) for f in _included(f, {f})} - {"ff8_launch.hpp"}
    assert used == files
    # a GEMM stage runs the kernel that small_gemm_tile chooses: that choice and both kernels count
    if bench.STAGE_SOURCE[stage] == "gemm.hip":
        assert {"gemm.hip", "gemm_small.hip", "gemm_rule.hpp"} <= files
