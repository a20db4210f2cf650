"""The build refuses kernels that spill registers where a spill costs time (host code, nothing is compiled here)."""
import glob
import os
import re

import pytest

from paper_2105_14450_amd import build

ASM = sorted(glob.glob(os.path.join(build.HERE, "_build", "gemm_edge_*-hip-amdgcn-amd-amdhsa-gfx950.s")))


def test_any_size_kernels_may_not_use_scratch_memory():
    assert build.scratch_limit("_ZN6cube3d4edge16gemm_edge_kernelINS0_4Bf16ELi128ELi2ELb1ELb0EEEvNS0_6ParamsE") == 0
    assert build.scratch_limit("_ZN6cube3d3mfk16gemm_mfma_kernelIvEEvv") == build.SCRATCH_LIMIT


@pytest.mark.skipif(not ASM, reason="no assembly of a build here")
def test_any_size_kernels_use_no_scratch_memory():
    seen = 0
    for path in ASM:
        with open(path) as f:
            text = f.read()
        for name, size in re.findall(r"\.name: +(\S*gemm_edge_kernel\S*)\n(?:.*\n)*? *\.private_segment_fixed_size: (\d+)", text):
            seen += 1
            assert int(size) == 0, name
    assert seen == 69
