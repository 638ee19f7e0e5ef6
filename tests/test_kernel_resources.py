"""What the compiled kernels take of a compute unit, as the library's own code objects state it: where a comment or a dispatch
rule counts on two workgroups in a unit at once, registers and LDS have to leave room for two.  Runs without a GPU."""
import os
import re
import struct
import subprocess

import pytest

from paper_2504_03702_amd import binding, build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
UNIT_VGPRS, UNIT_LDS = 512, 160 * 1024          # registers of a SIMD's lane (four SIMDs a unit), bytes of LDS
FIELDS = ("vgpr_count", "sgpr_spill_count", "vgpr_spill_count", "group_segment_fixed_size", "max_flat_workgroup_size")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: {field: value}} of the library."""
    if not os.path.exists(binding.LIB_PATH):
        build.build_library(verbose=False)
    tmp = tmp_path_factory.mktemp("objects")
    fat = str(tmp / "fatbin")
    subprocess.check_call([os.path.join(LLVM, "llvm-objcopy"), f"--dump-section=.hip_fatbin={fat}", binding.LIB_PATH,
                           str(tmp / "copy.so")])
    raw, found = open(fat, "rb").read(), {}
    for start in (m.start() for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", raw)):
        count, at = struct.unpack_from("<Q", raw, start + 24)[0], start + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", raw, at)
            target = raw[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in target or size == 0:
                continue
            path = str(tmp / "object")
            with open(path, "wb") as f:
                f.write(raw[start + offset:start + offset + size])
            notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], capture_output=True, text=True,
                                   check=True).stdout
            for part in notes.split("  - .agpr_count:")[1:]:
                name = subprocess.run(["c++filt", re.search(r"\.symbol:\s+'?(\S+?)\.kd", part).group(1)], capture_output=True,
                                      text=True, check=True).stdout
                name = re.sub(r"\(anonymous namespace\)::|^void ", "", name.strip())
                found[re.sub(r">\(.*|\(.*", lambda m: ">" if m.group().startswith(">") else "", name)] = {
                    k: int(re.search(rf"\.{k}:\s+(\d+)", part).group(1)) for k in FIELDS}
    return found


def workgroups_a_unit(k):
    """Workgroups of this kernel that registers and LDS let into a unit (registers are handed out by eights)."""
    waves = k["max_flat_workgroup_size"] // 64
    by_registers = UNIT_VGPRS // (-(-k["vgpr_count"] // 8) * 8) * 4 // waves
    return min(by_registers, UNIT_LDS // max(k["group_segment_fixed_size"], 1))


def test_maps_in_tiles_of_128_rows_leave_room_for_two(kernels):
    small = {n: k for n, k in kernels.items() if n.startswith("gemm_bf16_kernel<128")}
    assert any("true>" in n for n in small)                      # those that carry the maps of a few requests among them
    assert {n: workgroups_a_unit(k) for n, k in small.items() if workgroups_a_unit(k) < 2} == {}
    assert {n: k for n, k in small.items() if k["vgpr_spill_count"]} == {}


def test_short_router_calls_keep_their_scalars(kernels):
    """A decision is a chain of some 150 instructions, so scalars that do not fit their registers are paid for by every request of
    a call of few (19 of them: 2 to 3 % of 3 to 11 requests)."""
    few = {n: k for n, k in kernels.items() if re.match(r"route_kernel<[124], false", n)}
    assert few and {n: k for n, k in few.items() if k["sgpr_spill_count"] > 10 or k["vgpr_spill_count"]} == {}


def test_layer_norms_of_narrow_rows_spread_over_the_units(kernels):
    """Rows of 128 to 256 floats: eight to a workgroup, all of a row in registers (32 to a workgroup and a trip to memory for each
    pass made calls of some 1500 rows 3 % slower than a wavefront a row)."""
    narrow = {n: k for n, k in kernels.items() if re.match(r"layernorm_f32_narrow_kernel<[48]", n)}
    assert len(narrow) == 2
    assert {n: k for n, k in narrow.items() if k["max_flat_workgroup_size"] != 64 or k["vgpr_spill_count"] or k["sgpr_spill_count"]} == {}
