"""The rules by which a call takes one route or another, asked of the library's own headers at sizes where both sides have been
measured: a call keeps to the route that was the faster one there.  Runs without a GPU."""
import os
import subprocess

import pytest

from tests.test_host_sanitizers import CSRC, ROOT


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("dispatch") / "rules")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "dispatch", "rules.cpp"),
                           "-o", out])

    def run(rule, *numbers):
        line = " ".join([rule, *map(str, numbers)]) + "\n"
        return int(subprocess.run([out], input=line, capture_output=True, text=True, check=True).stdout)
    return run


def rows_of(tokens, n_req):
    """Rows of the workspace of a call: every request to whole eights, the last key tile's slack, whole 256s."""
    return -(-(tokens + 7 * n_req + 64) // 256) * 256


@pytest.mark.parametrize("hidden,n,length,padded,small", [
    # padded calls: eight or seven full rows of 512 slots through wide encoders (four layers, small / large: hidden 1024 872 /
    # 672 us; 2048 2835 / 1780 and 2364 / 1445), which narrow ones take in small tiles (768, half full 385 / 414)
    (1024, 8, 512, True, False), (2048, 8, 512, True, False), (2048, 7, 512, True, False), (768, 8, 512, True, True),
    (256, 8, 512, True, True), (768, 9, 512, True, False), (1024, 7, 512, True, True), (2048, 6, 512, True, True),
    # packed ones: up to 1536 rows whatever the width (hidden 2048, 16 of 56 tokens 788 / 877 us, 6 of 200 855 / 890)
    (2048, 16, 56, False, True), (2048, 6, 200, False, True), (2048, 6, 250, False, False), (1024, 6, 300, False, True),
    (1024, 6, 450, False, False), (768, 16, 150, False, True), (768, 16, 206, False, False), (256, 16, 206, False, True),
    (256, 16, 225, False, False), (256, 17, 20, False, False),
])
def test_small_tiles_where_they_are_faster(ask, hidden, n, length, padded, small):
    assert ask("small_maps", rows_of(n * length, n), int(padded), n, hidden) == small


@pytest.mark.parametrize("hidden,n,length,carried", [
    # where the launches of all rows' maps have idle units for the per-request tiles (prompts of 8 tokens, three layers, carried /
    # apart: hidden 1024 600 requests 919 / 954 us, 700 1086 / 1061, of 35 2173 / 2214; 2048 300 1612 / 1701, 400 1922 / 1897, 1000 4252 / 3973)
    (1024, 600, 8, True), (1024, 700, 8, False), (1024, 700, 35, True), (1280, 500, 8, False), (1280, 500, 35, True), (2048, 300, 8, True), (2048, 400, 8, False), (2048, 1000, 35, False),
    (1536, 400, 8, True), (1536, 700, 8, False), (768, 1024, 100, True), (256, 1024, 30, True), (512, 1025, 30, False),
    (768, 17, 30, True), (768, 16, 206, True), (768, 8, 20, False),
])
def test_side_maps_are_carried_where_that_is_faster(ask, hidden, n, length, carried):
    assert ask("carries_side_maps", rows_of(n * length, n), 0, n, hidden) == carried
