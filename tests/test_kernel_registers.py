"""Registers of the built kernels whose grids or plans assume how many workgroups fit a compute unit (512 registers per SIMD lane): four of
the split-K epilogue kernel, of four waves each, at most 128; two of the attention kernel, at most 256; neither keeps anything in scratch
memory.  Of the pipelined GEMM two workgroups of four waves at four to nine row tiles, but for the form that sums its slices inside the
launch, and one of eight, at most 256; the small-step GEMM's sixteen waves, at most 128."""
import os
import re
import shutil
import subprocess

import pytest

BUILD = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_05894_amd", "_build")
LLVM = "/opt/rocm/llvm/bin"


def kernels(source, tmp_path):
    """{mangled name: (registers, spilled registers, scratch bytes)} of the object built from `source`.hip."""
    obj = os.path.join(BUILD, source + ".o")
    if not os.path.exists(obj) or not os.path.exists(os.path.join(LLVM, "llvm-readelf")):
        pytest.skip("needs the built objects and the ROCm LLVM tools")
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    copy = shutil.copy(obj, str(tmp_path / "obj.o"))
    subprocess.run([LLVM + "/llvm-objcopy", "--dump-section", ".hip_fatbin=" + bundle, copy], check=True)
    subprocess.run([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    "--input=" + bundle, "--output=" + code], check=True)
    notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    found = {}
    for entry in re.split(r"\n  - \.a", notes)[1:]:      # one entry per kernel, its keys in alphabetical order
        field = lambda key: re.search(r"\." + key + r":\s+(\S+)", entry).group(1)
        found[field("symbol")] = tuple(int(field(key)) for key in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size"))
    return found


@pytest.mark.parametrize("source,name,count,most", [("stream_gemm", "epi_kernel", 5, 128), ("attention", "attn_partial_kernel", 14, 256)])
def test_registers_leave_room_for_the_workgroups_the_launch_assumes(source, name, count, most, tmp_path):
    mine = {k: v for k, v in kernels(source, tmp_path).items() if name in k}
    assert len(mine) == count, sorted(mine)
    for k, (registers, spilled, scratch) in mine.items():
        assert registers <= most and spilled == 0 and scratch == 0, (k, registers, spilled, scratch)


def test_registers_of_the_gemm_kernels(tmp_path):
    found = kernels("stream_gemm", tmp_path)
    small = {k: v for k, v in found.items() if "pgemm_kernel" in k}
    large = {tuple(int(x) for x in re.search(r"qgemm16_kernelILi(\d+)ELi(\d+)ELb(\d)ELi(\d)E", k).groups()): v for k, v in found.items() if "qgemm16_kernel" in k}
    assert len(small) == 112 and len(large) == 63
    for k, (registers, _, scratch) in small.items():
        # 8B and 70B QKV: the row scales' sums beside the first two tiles
        assert registers <= 128 and scratch <= (32 if "ILi0ELi8ELb0E" in k else 0), (k, registers, scratch)
    spilled = {(0, 8, 1, 2): 20, (9, 4, 0, 0): 20, (9, 4, 0, 1): 28}   # bytes of scratch a lane: blocks of eight and six tiles; nine tiles, two workgroups
    for (tiles, waves, blocks, form), (registers, _, scratch) in large.items():
        limit = 256 if waves == 8 or (4 <= tiles <= 9 and form != 2) else 512
        assert registers <= limit and scratch <= spilled.get((tiles, waves, blocks, form), 0), (tiles, waves, blocks, form, registers, scratch)
