"""The ring kernel of the any-size product: every tile, operand layout and element type at contractions of one K-tile, of
fewer K-tiles than the ring has stages, just above and below whole K-tiles and beyond the 64 that are looked up at a
time; several tiles per workgroup; shards that end inside a K-tile.  Integers in [-4, 4]: all sums are exact (below
2^24), so results are compared bit for bit with torch's fp32 product."""
import os
import subprocess

import pytest
import torch

import paper_2105_14450_amd as c3
from paper_2105_14450_amd import build

import gpu_util as gu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODES = {"f32": (torch.float32, c3.F32), "bf16": (torch.bfloat16, c3.BF16), "fp8_e4m3": (torch.float8_e4m3fn, c3.FP8_E4M3)}
LAYOUT = {c3.FORM_AB: (1, 0), c3.FORM_ABT: (1, 1), c3.FORM_ATB: (0, 0)}
# rows, columns, blocks per side of the cube, and contractions; multiples of 16 wherever an operand may be contiguous there
SIZES = [(48, 1040, 1, (272, 1040, 2064)), (816, 1040, 1, (400, 1040)), (400, 1040, 1, (144, 1040, 8208)), (1616, 2064, 1, (272, 400, 1040)),
         (2064, 4112, 1, (2064,)), (4112, 2064, 1, (1040, 2064)), (4112, 4112, 1, (80, 1040)), (272, 144, 3, (1040,)),
         (3088, 1168, 1, (1040, 4624)), (1136, 7152, 1, (1040, 4112)), (2064, 3088, 1, (4112,))]
CASES = [(dtype, out, form) for dtype, out in (("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32"), ("fp8_e4m3", "bf16"), ("fp8_e4m3", "f32"))
         for form in LAYOUT]


def _integers(shape, gen):
    return torch.randint(-4, 5, shape, device="cuda", generator=gen, dtype=torch.int8).float()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,out,form", CASES)
def test_ring_tiles(dtype, out, form):
    storage, code = CODES[dtype]
    gen = torch.Generator(device="cuda").manual_seed(form)
    for m, n, q, contractions in SIZES:
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
@pytest.mark.gpu
@pytest.mark.parametrize("form", LAYOUT)
@pytest.mark.parametrize("m,n,k", [(1616, 2064, 1040), (1136, 7152, 4112), (4112, 2064, 2064)])
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
@pytest.mark.gpu
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


# q = 3: blocks of 3 shards that end inside a K-tile (of 64 to 256 indices), in every direction; a bias with the forward
@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(9 * 272, 3 * 656, 9 * 368), (9 * 304, 3 * 272, 9 * 272), (9 * 16, 3 * 1040, 9 * 272)])
@pytest.mark.parametrize("dtype", sorted(CODES))
def test_ring_in_place(dtype, M, K, N):
    q, (storage, code) = 3, CODES[dtype]
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


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="ROCm compiler not found")
def test_sizes_reach_every_tile(tmp_path):
    c3.binding.load()
    exe = str(tmp_path / "ring_plan")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-I", build.INCLUDE, "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "host", "ring_plan.cpp"), "-x", "none", build.LIB,
                    "-Wl,-rpath," + os.path.dirname(build.LIB), "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True, capture_output=True)
    asked = [(case, (m, n, q, k)) for case in CASES for m, n, q, ks in SIZES for k in ks]
    lines = ["%d %d %d %d %d %d %d %d" % (CODES[t][1], CODES[o][1], *LAYOUT[f], q ** 3, m, n, k) for (t, o, f), (m, n, q, k) in asked]
    res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True, timeout=60)
    reached = {(case, tuple(map(int, line.split()))) for (case, _), line in zip(asked, res.stdout.splitlines())}
    tiles = lambda dtype: ((64, 64), (128, 128)) if dtype == "f32" else ((32, 32), (64, 64), (128, 128), (128, 256), (256, 128))
    missing = {(case, tile) for case in CASES for tile in tiles(case[0])} - reached
    assert not missing, sorted(missing)
