"""The ring kernel of the any-size product: every tile, operand layout and element type at contractions of one K-tile, of
fewer K-tiles than the ring has stages, just above and below whole K-tiles and beyond the 64 that are looked up at a
time; several tiles per workgroup; results with streaming stores and element by element; shards that end inside a K-tile;
operands at the limit of its addresses.  (That the sizes reach all this is asserted in test_product_dispatch.py.)
Integers in [-4, 4]: all sums are exact (below 2^24), so results are compared bit for bit with torch's fp32 product."""
import pytest
import torch

import paper_2105_14450_amd as c3

import gpu_util as gu
import product_shapes as ps

CODES = {"f32": (torch.float32, c3.F32), "bf16": (torch.bfloat16, c3.BF16), "fp8_e4m3": (torch.float8_e4m3fn, c3.FP8_E4M3)}
LAYOUT = {c3.FORM_AB: (1, 0), c3.FORM_ABT: (1, 1), c3.FORM_ATB: (0, 0)}
CASES = [(dtype, out, form) for dtype, out in (("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32"), ("fp8_e4m3", "bf16"), ("fp8_e4m3", "f32"))
         for form in LAYOUT]

pytestmark = pytest.mark.gpu


def _integers(shape, gen):
    return torch.randint(-4, 5, shape, device="cuda", generator=gen, dtype=torch.int8).float()


@pytest.mark.parametrize("dtype,out,form", CASES)
def test_ring_tiles(dtype, out, form):
    storage, code = CODES[dtype]
    gen = torch.Generator(device="cuda").manual_seed(form)
    for m, n, q, contractions in ps.RING + ps.RING_LINES + (ps.RING_ODD if form == c3.FORM_ABT else []):
        for k in contractions:
            a, b = _integers((q ** 3, m, k), gen), _integers((q ** 3, k, n), gen)
            left = (a.transpose(1, 2) if form == c3.FORM_ATB else a).contiguous().to(storage)
            right = (b.transpose(1, 2) if form == c3.FORM_ABT else b).contiguous().to(storage)
            mm = c3.make_matmul(q, form, m, n, k, in_dtype=code, out_dtype=CODES[out][1])
            got = torch.full((q ** 3, m, n), float("nan"), device="cuda", dtype=CODES[out][0])
            c3.cube3d_matmul_blocks(mm, left, right, got)
            assert torch.equal(got, torch.bmm(a, b).to(got.dtype)), "%d x %d x %d" % (m, n, k)


# fp8: tiles of 128 and more take the 64-deep MFMA for bf16 results, smaller ones and fp32 results the shallower ones.  A row's
# bits do not depend on that: a call with bf16 results is one with fp32 results rounded once, and the rows of a call with
# few rows are those of one with many.  Random bytes, whose sums depend on the order in nearly every element; against 64 bits
# one rounding to bf16 and 1e-4 of the largest entry for the matrix cores' sums.
@pytest.mark.parametrize("form", LAYOUT)
@pytest.mark.parametrize("m,n,k", ps.RING_DEEP)
def test_fp8_bits_do_not_depend_on_the_tile(m, n, k, form):
    gen = torch.Generator(device="cuda").manual_seed(m + form)

    def codes(rows, cols):      # every one but the two NaNs
        t = torch.randint(0, 254, (rows, cols), device="cuda", generator=gen, dtype=torch.int16)
        return (t + (t >= 127)).to(torch.uint8)

    def product(rows, out):
        left = (a[:rows].t() if form == c3.FORM_ATB else a[:rows]).contiguous().view(torch.float8_e4m3fn)
        right = (b.t() if form == c3.FORM_ABT else b).contiguous().view(torch.float8_e4m3fn)
        mm = c3.make_matmul(1, form, rows, n, k, in_dtype=c3.FP8_E4M3, out_dtype=CODES[out][1])
        got = torch.full((rows, n), float("nan"), device="cuda", dtype=CODES[out][0])
        c3.cube3d_matmul_blocks(mm, left, right, got)
        return got

    a, b = codes(m, k), codes(k, n)
    got = product(m, "bf16")
    for rows in (400, 48):
        assert torch.equal(product(rows, "bf16"), got[:rows]), rows
    assert torch.equal(product(m, "f32").to(torch.bfloat16), got)
    want = a.view(torch.float8_e4m3fn).double() @ b.view(torch.float8_e4m3fn).double()
    bound = want.abs() / 256 + 1e-4 * want.abs().max()
    assert bool(((got.double() - want).abs() <= bound).all())


# Tile-aligned fp8 products run on the tuned kernel with many rows and on the ring with few: the same bits too (no split of
# the contraction at these sizes).  Random bytes; plain operands and a cube of one processor read in place.
@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("form", LAYOUT)
def test_fp8_bits_of_few_and_many_aligned_rows(form, out):
    gen = torch.Generator(device="cuda").manual_seed(form)
    m, n, k = 16384, 1024, 1024
    t = torch.randint(0, 254, (m + n, k), device="cuda", generator=gen, dtype=torch.int16)
    t = (t + (t >= 127)).to(torch.uint8)
    a, b = t[:m], t[m:].t()
    plain, in_place = {}, {}
    for rows in (m, 256):
        left = (a[:rows].t() if form == c3.FORM_ATB else a[:rows]).contiguous().view(torch.float8_e4m3fn)
        right = (b.t() if form == c3.FORM_ABT else b).contiguous().view(torch.float8_e4m3fn)
        mm = c3.make_matmul(1, form, rows, n, k, in_dtype=c3.FP8_E4M3, out_dtype=CODES[out][1])
        assert c3.cube3d_matmul_workspace_bytes(mm) == 0
        plain[rows], in_place[rows] = (torch.full((rows, n), float("nan"), device="cuda", dtype=CODES[out][0]) for _ in range(2))
        c3.cube3d_matmul_blocks(mm, left, right, plain[rows])
        x, y, z = c3.AXIS_X, c3.AXIS_Y, c3.AXIS_Z
        stored = lambda shape, code: c3.make_matrix(1, *shape, x, y, c3.SPLIT_ROWS, code)
        c3.virtual_cube_matmul(form, stored(left.shape, c3.FP8_E4M3), stored(right.shape, c3.FP8_E4M3), stored((rows, n), CODES[out][1]),
                               left, right, in_place[rows], 1.0, 1.0)
        assert torch.equal(plain[rows], in_place[rows]), rows
    assert torch.equal(plain[m][:256], plain[256])


# shards that end inside a K-tile, of whole cache lines, of an odd number of columns; a bias with the forward
@pytest.mark.parametrize("q,M,K,N", ps.RING_CUBES + ps.RING_CUBES_LINES + ps.RING_CUBES_ODD)
@pytest.mark.parametrize("dtype", sorted(CODES))
def test_ring_in_place(dtype, q, M, K, N):
    storage, code = CODES[dtype]
    result = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(M)
    X, W, G, bias = _integers((M, K), gen), _integers((K, N), gen), _integers((M, N), gen), _integers((N,), gen)
    d = c3.make_desc(q, M, K, N, in_dtype=code, out_dtype=c3.F32)
    x, w, g = (gu.device_shards(t, name, q).to(storage) for t, name in ((X, "x"), (W, "w"), (G, "y")))
    diagonal = torch.zeros((q ** 3, N // q ** 2), device="cuda")
    c3.virtual_cube_scatter(d, c3.OPERAND_BIAS, bias, diagonal)
    y, dx, dw = (torch.full(t.shape, float("nan"), device="cuda", dtype=result) for t in (g, x, w))
    c3.virtual_cube_linear_fwd(d, x, w, diagonal, y)
    c3.virtual_cube_linear_bwd_dx(d, g, w, dx)
    c3.virtual_cube_linear_bwd_dw(d, x, g, dw)
    for got, want, name in ((y, X @ W + bias, "y"), (dx, G @ W.t(), "x"), (dw, X.t() @ G, "w")):
        assert torch.equal(got, gu.device_shards(want, name, q).to(result)), name


# An operand of 1 GiB at most is addressed through a buffer of that size, whose end marks rows and indices beyond the edges.
@pytest.mark.parametrize("above", [False, True])
@pytest.mark.parametrize("dtype", sorted(ps.ONE_GB))
def test_operands_around_1_gb(dtype, above):
    storage, code = CODES[dtype]
    cols, n, rows = ps.ONE_GB[dtype][0], 16, ps.ONE_GB[dtype][2 if above else 1]
    gen = torch.Generator(device="cuda").manual_seed(rows)
    large, wide, tall = _integers((rows, cols), gen), _integers((cols, n), gen), _integers((rows, n), gen)
    stored = large.to(storage)
    for form, right, shape, want in ((c3.FORM_AB, wide, (rows, n, cols), large @ wide),
                                     (c3.FORM_ABT, wide.t().contiguous(), (rows, n, cols), large @ wide),
                                     (c3.FORM_ATB, tall, (cols, n, rows), large.t() @ tall)):
        mm = c3.make_matmul(1, form, *shape, in_dtype=code, out_dtype=c3.F32)
        got = torch.full(shape[:2], float("nan"), device="cuda")
        c3.cube3d_matmul_blocks(mm, stored, right.to(storage), got)
        assert torch.equal(got, want), "form %d" % form
