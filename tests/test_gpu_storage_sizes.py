"""Scatter and assemble (GPU) at both sides of the size from which they write with streaming stores: 128 MiB each way.
Copies, compared bit for bit with index arithmetic on the device."""
import pytest
import torch

import paper_2105_14450_amd as c3

import gpu_util as gu

pytestmark = pytest.mark.gpu

Q = 2
WHICH = {"x": (c3.OPERAND_X, c3.OPERAND_DX), "w": (c3.OPERAND_W, c3.OPERAND_DW), "y": (c3.OPERAND_DY, c3.OPERAND_Y)}


@pytest.mark.parametrize("operand", ["x", "w", "y"])
@pytest.mark.parametrize("rows,cols", [(8192, 8192), (8196, 8192), (16384, 8192), (8196, 8204)])
def test_storage_round_trip(operand, rows, cols):
    M, K, N = {"x": (rows, cols, 4), "w": (4, rows, cols), "y": (rows, 2, cols)}[operand]
    d = c3.make_desc(Q, M, K, N, in_dtype=c3.BF16, out_dtype=c3.F32, shard_dtype=c3.BF16)
    gen = torch.Generator(device="cuda").manual_seed(rows)
    full = torch.randint(-2 ** 15, 2 ** 15, (rows, cols), device="cuda", generator=gen, dtype=torch.int16)
    want = gu.device_shards(full, operand, Q)
    got, back = torch.zeros_like(want), torch.zeros_like(full)
    c3.virtual_cube_scatter(d, WHICH[operand][0], full, got)
    c3.virtual_cube_assemble(d, WHICH[operand][1], want, back)
    assert torch.equal(got, want) and torch.equal(back, full)
