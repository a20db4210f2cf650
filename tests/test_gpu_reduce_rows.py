"""Reduce-scatters with one row per wavefront (few rows, or long ones) and with four (many short rows): row counts that are no
multiple of a workgroup's, in 16-byte and in single pieces, one step of a row and several.  Integers: every sum is exact, so the
result is compared bit for bit with torch's."""
import pytest
import torch

import paper_2105_14450_amd as c3

pytestmark = pytest.mark.gpu

CODES = {"f32": (torch.float32, c3.F32), "bf16": (torch.bfloat16, c3.BF16)}


# q = 2: rows and lengths M/4 x N/2 (Y), M/4 x K/2 (dX), K/2 x N/4 (dW); 8 processors, so four rows each where
# rows are more than 512 times the steps of 256 (lengths divisible by 4) or 64 elements
@pytest.mark.parametrize("M,K,N", [(4, 2, 4), (4 * 13, 2 * 9, 4 * 67), (4 * 512, 2 * 513, 4 * 64), (4 * 515, 2 * 517, 4 * 33),
                                   (4 * 1027, 2 * 1031, 4 * 5), (4 * 1026, 2 * 1100, 4 * 258), (4 * 4093, 2 * 4099, 4 * 8)])
@pytest.mark.parametrize("partial,shard", [("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16")])
def test_rows_per_wavefront(M, K, N, partial, shard):
    q, gen = 2, torch.Generator(device="cuda").manual_seed(M)
    d = c3.make_desc(q, M, K, N, in_dtype=c3.BF16, out_dtype=CODES[partial][1], shard_dtype=CODES[shard][1])
    part = lambda *s: torch.randint(-64, 65, (q, q, q) + s, device="cuda", generator=gen, dtype=torch.int8).to(CODES[partial][0])
    bias = torch.randint(-64, 65, (q ** 3, N // q), device="cuda", generator=gen, dtype=torch.int8).float()
    P, Q, R = part(M // q, N // q), part(M // q, K // q), part(K // q, N // q)
    Ms, Ns = M // 4, N // 4
    y = P.float().sum(2).view(q, q, q, Ms, N // q)
    dx = Q.float().sum(1).view(q, q, q, Ms, K // q).transpose(1, 2)
    dw = R.float().sum(0).view(q, q, K // q, q, Ns).permute(3, 0, 1, 2, 4)
    new = lambda like: torch.full((q ** 3,) + like.shape[3:], float("nan"), device="cuda", dtype=CODES[shard][0])
    got = [new(t) for t in (y, y, dx, dw)]
    c3.virtual_cube_reduce_scatter(d, c3.OPERAND_Y, c3.AXIS_Z, P, got[0])
    c3.virtual_cube_reduce_scatter_bias(d, c3.AXIS_Z, P, bias, got[1])
    c3.virtual_cube_reduce_scatter(d, c3.OPERAND_DX, c3.AXIS_Y, Q, got[2])
    c3.virtual_cube_reduce_scatter(d, c3.OPERAND_DW, c3.AXIS_X, R, got[3])
    for t, want, name in zip(got, (y, y + bias.view(q, q, q, 1, N // q), dx, dw), ("Y", "Y + b", "dX", "dW")):
        assert torch.equal(t, want.reshape(t.shape).to(t.dtype)), name
