"""Register and LDS budget of the large-tile (bf16 and UE8M0 fp8) and
wide-tile stage-2 GEMMs, from the compiler's kernel metadata (CPU only: hipcc
cross-compiles for gfx950).

The kernels stream their operands with LDS DMA issued from inline assembly,
which the compiler does not track; a register spill makes it wait for every
vector-memory load in flight before the reload, which drains the DMA ring.
So they must compile without spills, and their rings must fit the 160 KB
of LDS of a gfx950 CU.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2608_13057_amd import build

SOURCES = {"bf16": os.path.join(build.CSRC, "gemm_big_agpr.hip"), "fp8": os.path.join(build.CSRC, "gemm_big_f8_agpr.hip")}


def _metadata(tmp_path, SRC):
    if not os.path.exists(build.HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = tmp_path / "big.s"
    cmd = [build.HIPCC, *build.flags_for(SRC), "-Wno-inline-asm", "--cuda-device-only", "-S", SRC, "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    text = out.read_text()
    kernels = {}
    # the metadata lists one block per kernel: ".name: <symbol>" with its
    # resource fields around it
    for block in text.split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        fields = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", block)}
        kernels[name] = fields
    return kernels


@pytest.mark.parametrize("which", sorted(SOURCES))
def test_large_tile_gemm_has_no_spills_and_fits_lds(tmp_path, which):
    kernels = _metadata(tmp_path, SOURCES[which])
    big = {n: f for n, f in kernels.items() if "k_gemm_big" in n}
    assert len(big) == 2, sorted(kernels)  # gate/up and down
    for name, f in big.items():
        assert f["vgpr_spill_count"] == 0, (name, f)
        # scalar spills go to lanes of a VGPR (v_writelane / v_readlane), no
        # memory access; the bf16 kernel has none, the fp8 one several dozen
        # (its DMA cursor keeps the next item's bases and per-piece offsets
        # in scalar registers; the spilled values are read per item, not
        # per sub-step)
        assert f["sgpr_spill_count"] <= (0 if which == "bf16" else 96), (name, f)
        assert f["group_segment_fixed_size"] <= 160 * 1024, (name, f)
        assert f.get("private_segment_fixed_size", 0) == 0, (name, f)


def test_wide_tile_gemm_has_no_spills_and_fits_lds(tmp_path):
    kernels = _metadata(tmp_path, os.path.join(build.CSRC, "gemm_wide.hip"))
    wide = {n: f for n, f in kernels.items() if "k_gemm_wide" in n}
    assert len(wide) == 6, sorted(kernels)  # three element types, gate/up and down
    for name, f in wide.items():
        assert f["vgpr_spill_count"] == 0, (name, f)
        assert f["vgpr_count"] <= 256, (name, f)  # two wavefronts per SIMD
        # to lanes of a VGPR, read per item (29 .. 70 of them)
        assert f["sgpr_spill_count"] <= 96, (name, f)
        assert f["group_segment_fixed_size"] <= 160 * 1024, (name, f)
        assert f.get("private_segment_fixed_size", 0) == 0, (name, f)
