"""The bench reports counted traffic only for the sources it was counted on: all of the GEMM kernel's have to be among them."""
import os
import re

import bench


def test_counted_traffic_is_tied_to_all_sources_of_the_gemm():
    csrc = os.path.join(bench.ROOT, "paper_2504_03702_amd", "csrc")
    todo, seen = ["gemm_bf16.hip"], set()
    while todo:
        name = todo.pop()
        if name in seen or not os.path.exists(os.path.join(csrc, name)):
            continue
        seen.add(name)
        with open(os.path.join(csrc, name)) as f:
            todo += re.findall(r'^#include "([^"]+)"', f.read(), flags=re.M)
    with open(os.path.join(csrc, "rowops.hip")) as f:
        assert "GemmPlan plan_gemm(" in f.read()                 # the heights of the tiles
    assert seen | {"rowops.hip"} == set(bench.GEMM_SOURCES)
