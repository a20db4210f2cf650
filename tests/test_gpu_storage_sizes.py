"""Scatter and assemble (GPU) at both sides of the size from which they write with streaming stores: 128 MiB each way.
Copies, compared bit for bit with index arithmetic on the device."""
import pytest
import torch

import paper_2105_14450_amd as c3

pytestmark = pytest.mark.gpu

Q = 2
# order of (i, a, b, rows of a shard, columns of a shard) in the full matrix: (row indices), (column indices)
ORDER = {"x": ((0, 1, 3), (2, 4)), "w": ((2, 3), (1, 0, 4)), "y": ((0, 2, 3), (1, 4))}
WHICH = {"x": (c3.OPERAND_X, c3.OPERAND_DX), "w": (c3.OPERAND_W, c3.OPERAND_DW), "y": (c3.OPERAND_DY, c3.OPERAND_Y)}


def shards(full, operand):
    order = [d for part in ORDER[operand] for d in part]
    cut = [s for n, part in zip(full.shape, ORDER[operand]) for s in [Q] * (len(part) - 1) + [n // Q ** (len(part) - 1)]]
    return full.reshape(cut).permute([order.index(d) for d in range(5)]).contiguous()


@pytest.mark.parametrize("operand", ["x", "w", "y"])
@pytest.mark.parametrize("rows,cols", [(8192, 8192), (8196, 8192), (16384, 8192), (8196, 8204)])
def test_storage_round_trip(operand, rows, cols):
    M, K, N = {"x": (rows, cols, 4), "w": (4, rows, cols), "y": (rows, 2, cols)}[operand]
    d = c3.make_desc(Q, M, K, N, in_dtype=c3.BF16, out_dtype=c3.F32, shard_dtype=c3.BF16)
    gen = torch.Generator(device="cuda").manual_seed(rows)
    full = torch.randint(-2 ** 15, 2 ** 15, (rows, cols), device="cuda", generator=gen, dtype=torch.int16)
    want = shards(full, operand)
    got, back = torch.zeros_like(want), torch.zeros_like(full)
    c3.virtual_cube_scatter(d, WHICH[operand][0], full, got)
    c3.virtual_cube_assemble(d, WHICH[operand][1], want, back)
    assert torch.equal(got, want) and torch.equal(back, full)
