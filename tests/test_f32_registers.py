"""Registers of the float32 attention kernel, from the compiler's own listing (no GPU): no instance spills, and those of D = 64 leave
room for the wavefronts per SIMD that their calls with many workgroups live on. (A second K/V register set cost a wavefront per SIMD
and spilled at D = 128: 32 requests x 32 heads of 100 keys, trees of 8, us, one set / two: 35.2 / 39.5, D = 64 19.4 / 22.7.)"""
import os
import re
import subprocess

import pytest

from paper_2305_09781_amd import build

# D, query tiles: wavefronts per SIMD (512 VGPRs, taken by eights)
WAVES = {("128", "1"): 2, ("64", "1"): 4, ("64", "2"): 3, ("128", "2"): 2}


def test_float32_instances_do_not_spill(tmp_path):
    try:
        hipcc = build._hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    asm = tmp_path / "f32.s"
    subprocess.run([hipcc, *build.HIPCC_FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "tree_attention_f32.hip"), "-o", str(asm)],
                   check=True, capture_output=True)
    seen = {}
    for block in asm.read_text().split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        m = re.search(r"tree_attention_f32_kernelILi(\d+)ELi(\d+)ELb(\d)E", name)
        if m:
            seen[m.groups()] = {k: int(re.search(r"\.%s:\s+(\d+)" % k, block).group(1))
                                for k in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    assert len(seen) == 8
    for (D, tiles, append), r in seen.items():
        assert r["vgpr_spill_count"] == 0 and r["private_segment_fixed_size"] == 0, (D, tiles, append, r)
        assert 512 // (-(-r["vgpr_count"] // 8) * 8) >= WAVES[D, tiles], (D, tiles, append, r)
