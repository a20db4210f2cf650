"""The build refuses kernels that spill registers where a spill costs time (host code, nothing is compiled here)."""
import glob
import os
import re

import pytest

from paper_2105_14450_amd import build

ALL_ASM = sorted(glob.glob(os.path.join(build.HERE, "_build", "*-hip-amdgcn-amd-amdhsa-gfx950.s")))


def test_any_size_kernels_may_not_use_scratch_memory():
    assert build.scratch_limit("_ZN6cube3d4edge16gemm_edge_kernelINS0_4Bf16ELi128ELi2ELb1ELb0EEEvNS0_6ParamsE") == 0
    assert build.scratch_limit("_ZN6cube3d4edge16gemm_ring_kernelINS0_4Bf16ELi256ELi128ELi3ELb1ELb1ELb0EEEvNS0_6ParamsE") == 0
    assert build.scratch_limit("_ZN6cube3d3mfk16gemm_mfma_kernelIvEEvv") == build.SCRATCH_LIMIT


@pytest.mark.skipif(not ALL_ASM, reason="no assembly of a build here")
def test_any_size_kernels_use_no_scratch_memory():
    seen = {"gemm_edge_kernel": 0, "gemm_ring_kernel": 0}
    for path in ALL_ASM:
        with open(path) as f:
            text = f.read()
        for name, kind, size in re.findall(r"\.name: +(\S*(gemm_edge_kernel|gemm_ring_kernel)\S*)\n(?:.*\n)*? *\.private_segment_fixed_size: (\d+)", text):
            seen[kind] += 1
            assert int(size) == 0, name
    assert seen == {"gemm_edge_kernel": 69, "gemm_ring_kernel": 63}


LOAD = "\tglobal_load_lds_dwordx4 v1, s[44:45]"


@pytest.mark.parametrize("lines,early", [
    (["v_readlane_b32 s45, v9, 3", "s_mov_b32 m0, s11", "s_nop 0"], True),
    (["v_readlane_b32 s45, v9, 3", "s_mov_b32 m0, s11", "s_nop 3"], False),
    (["v_readlane_b32 s46, v9, 3", "s_mov_b32 m0, s11", "s_nop 0"], False),
    (["v_readlane_b32 s45, v9, 3", "s_mov_b64 s[44:45], s[44:45]", "s_nop 0"], False),
    (["v_readfirstlane_b32 s44, v9", "s_mov_b32 s45, s46"], True),
    (["v_add_co_u32_e64 v3, s[44:45], v3, v4", "s_nop 3"], True),
    (["v_readlane_b32 s45, v9, 3", "s_cbranch_scc1 .LBB0_2", "s_nop 7", ".LBB0_2:"], True),
    (["s_branch .LBB0_2", "v_readlane_b32 s45, v9, 3", "s_branch .LBB0_3", ".LBB0_2:"], False)])
def test_scalar_registers_read_too_early_are_found(lines, early):
    asm = ["kernel:"] + ["\t" + x if not x.endswith(":") else x for x in lines] + [LOAD, "\ts_nop 7", ".LBB0_3:", "\ts_endpgm"]
    found = build.early_scalar_reads(x + "\n" for x in asm)
    assert bool(found) == early and all(name == "kernel" for name, _, _ in found)


@pytest.mark.skipif(not ALL_ASM, reason="no assembly of a build here")
def test_no_load_reads_a_scalar_register_too_early():
    for path in ALL_ASM:
        with open(path) as f:
            assert not build.early_scalar_reads(f), path
