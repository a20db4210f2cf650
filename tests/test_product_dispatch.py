"""Which kernel, tile and load width a product of any size runs on: the dispatch is host code, so it is asked on the
CPU (``tests/host/product_plan.cpp`` linked against the library; nothing is launched)."""
import collections
import os
import subprocess

import pytest

import paper_2105_14450_amd as c3
from paper_2105_14450_amd import build

import product_shapes as ps

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAYOUT = {c3.FORM_AB: (1, 0), c3.FORM_ABT: (1, 1), c3.FORM_ATB: (0, 0)}

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="ROCm compiler not found")


Route = collections.namedtuple("Route", "tile piece rows columns wide stream tuned")


@pytest.fixture(scope="session")
def routes(tmp_path_factory):
    """What product_plan.cpp prints, one Route per line asked."""
    c3.binding.load()
    exe = str(tmp_path_factory.mktemp("plan") / "product_plan")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-I", build.INCLUDE, "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "host", "product_plan.cpp"), "-x", "none", build.LIB,
                    "-Wl,-rpath," + os.path.dirname(build.LIB), "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True, capture_output=True)

    def ask(lines):
        res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True, timeout=60)
        return [Route(*map(int, line.split())) for line in res.stdout.splitlines()]
    return ask


@pytest.fixture(scope="session")
def plans(routes):
    """Tile side and load width of the any-size kernel (which the ring kernel takes in its place is not asked)."""
    return lambda lines: [tuple(r[:2]) for r in routes(lines)]


def plain(dtype, form, m, n, k, batch=1, out=c3.BF16):
    return "plain %d %d %d %d %d %d %d %d" % (dtype, out, *LAYOUT[form], batch, m, n, k)


def test_launches_stay_below_the_grid_limit(plans):
    # 64000 blocks of 1 x 33600: 2^24 tiles of 256 work-items and more do not fit one grid dimension, the element-wise
    # kernel has the batch in another one
    assert plans([plain(c3.BF16, form, 1, 33600, 1, batch=64000) for form in LAYOUT]) == [(0, 0)] * 3
    for tile, piece in plans([plain(c3.BF16, form, 8, 64, 4096, batch=64000) for form in LAYOUT]):
        assert tile and -(-8 // tile) * -(-64 // tile) * 64000 < 1 << 24


def cube(dtype, op, q, M, K, N, out=c3.BF16):
    return "cube %d %d %d %d %d %d %d" % (dtype, out, op, q, M, K, N)


# Short contractions: the element-wise kernel took 1.5 to 8 times less time than any tile on each of these; 1.1 times on the
# longest, in single bytes.
@pytest.mark.parametrize("line", [
    plain(c3.BF16, c3.FORM_ABT, 1, 5, 9, 4096), plain(c3.FP8_E4M3, c3.FORM_ABT, 1, 4, 5, 4096),
    plain(c3.BF16, c3.FORM_AB, 41, 41, 17, 4096), plain(c3.BF16, c3.FORM_AB, 40, 40, 16, 4096),
    plain(c3.FP8_E4M3, c3.FORM_AB, 41, 41, 97, 4096), plain(c3.FP8_E4M3, c3.FORM_AB, 101, 201, 129, 512),
    plain(c3.FP8_E4M3, c3.FORM_ABT, 8, 130, 66, 512), plain(c3.FP8_E4M3, c3.FORM_ATB, 3001, 3001, 257),
    plain(c3.BF16, c3.FORM_AB, 3001, 3001, 33), plain(c3.F32, c3.FORM_AB, 3001, 3001, 17, out=c3.F32),
    plain(c3.FP8_E4M3, c3.FORM_AB, 3001, 3001, 1025), plain(c3.BF16, c3.FORM_AB, 1001, 1001, 17), plain(c3.F32, c3.FORM_AB, 41, 41, 17, 4096, out=c3.F32)])
def test_short_contractions_run_element_by_element(plans, line):
    assert plans([line]) == [(0, 0)]


# Tiles that lie mostly beyond the output are not worth their time: 1.5 to 6 times as long with tiles of 128.
@pytest.mark.parametrize("line,tile", [
    (plain(c3.BF16, c3.FORM_AB, 41, 41, 1025, 4096), 64), (plain(c3.BF16, c3.FORM_AB, 9, 9, 1025, 4096), 32),
    (plain(c3.BF16, c3.FORM_AB, 40, 40, 512, 4096), 64), (plain(c3.F32, c3.FORM_AB, 40, 40, 512, 4096, out=c3.F32), 64),
    (plain(c3.FP8_E4M3, c3.FORM_ATB, 24, 24, 1024, 4096), 32), (plain(c3.BF16, c3.FORM_AB, 16, 256, 1024, 512), 64)])
def test_small_blocks_run_on_small_tiles(plans, line, tile):
    assert plans([line])[0][0] == tile


# Longer contractions stay on the tiles.
@pytest.mark.parametrize("line,want", [
    (plain(c3.BF16, c3.FORM_AB, 3000, 3000, 64), (128, 16)), (plain(c3.BF16, c3.FORM_AB, 1000, 1000, 128), (64, 16)),
    (plain(c3.F32, c3.FORM_AB, 128, 64, 64, 8, out=c3.F32), (32, 16)), (plain(c3.FP8_E4M3, c3.FORM_AB, 3001, 3001, 2049), (64, 1)),
    (plain(c3.BF16, c3.FORM_ABT, 1001, 1001, 513), (64, 2)), (cube(c3.BF16, 0, 4, 64, 2048, 8192), (32, 16)),
    (cube(c3.BF16, 2, 4, 64, 2048, 8192), (128, 16)), (cube(c3.FP8_E4M3, 1, 2, 3000, 3072, 12288), (128, 16)),
    (cube(c3.BF16, 2, 3, 2997, 1152, 4608), (128, 16))])
def test_longer_contractions_run_on_tiles(plans, line, want):
    assert plans([line]) == [want]


def _kernel(dtype, tile, piece):
    """The instantiation a plan runs on: (tile side, bytes per load)."""
    return tile, 16 if piece >= 16 else 4 if piece >= 4 else {c3.F32: 4, c3.BF16: 2, c3.FP8_E4M3: 1}[dtype]


NAMES = {"f32": c3.F32, "bf16": c3.BF16, "fp8_e4m3": c3.FP8_E4M3}
OPS = (c3.FORM_AB, c3.FORM_ABT, c3.FORM_ATB)        # operand layouts of forward, dX and dW


# The sizes of the GPU tests reach all 69 kernels through registers, those of a cube in place every one with tiles of 64 and
# 128.  What the ring kernel or the tile-aligned one takes does not count.
def test_gpu_tests_reach_every_kernel(routes):
    widths = {c3.BF16: (16, 4, 2), c3.FP8_E4M3: (16, 4, 1), c3.F32: (16, 4)}
    every = {(t, layout, tile, w) for t in widths for layout in LAYOUT.values() for tile in (32, 64, 128) for w in widths[t]
             if not (w == 1 and tile == 128)}
    assert len(every) == 69

    def run(asked):
        return {(t, LAYOUT[form], *_kernel(t, r.tile, r.piece)) for (t, form, _), r in zip(asked, routes([a[2] for a in asked]))
                if r.tile and not r.rows and not r.tuned}
    result = lambda t: c3.F32 if t == c3.F32 else c3.BF16
    plain_asked = [(t, form, plain(t, form, m, n, k, out=result(t))) for t in widths for form in LAYOUT for u in ps.OUTPUTS
                   for m, n in ps.OUTPUTS[u] for k in ps.CONTRACTIONS[u]]
    cubes = [(t, 3, sizes) for t in widths for u in ps.CUBES for sizes in ps.CUBES[u]]
    cubes += [(NAMES[name], 8, sizes) for name in ps.SHORT_SHARDS for sizes in ps.SHORT_SHARDS[name]]
    in_place = run([(t, OPS[op], cube(t, op, q, *sizes, out=result(t))) for t, q, sizes in cubes for op in range(3)])
    assert run(plain_asked) | in_place == every, every - run(plain_asked) - in_place
    assert in_place >= {x for x in every if x[2] > 32}, {x for x in every if x[2] > 32} - in_place


RING_TYPES = [(t, out) for t, out in (("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32"), ("fp8_e4m3", "bf16"), ("fp8_e4m3", "f32"))]


def _ring_tiles(dtype):
    return ((64, 64), (128, 128)) if dtype == "f32" else ((32, 32), (64, 64), (128, 128), (128, 256), (256, 128))


# The sizes of test_gpu_ring_product.py reach every tile in every type and layout, on both sides of what the kernel decides by
# the result: streaming stores (tiles above 128 x 128), elements one by one (A B^T on plain operands).
def test_gpu_tests_reach_every_ring_kernel(routes):
    asked = [((t, out, form), plain(NAMES[t], form, m, n, k, q ** 3, NAMES[out])) for t, out in RING_TYPES for form in LAYOUT
             for m, n, q, ks in ps.RING + ps.RING_LINES + (ps.RING_ODD if form == c3.FORM_ABT else []) for k in ks]
    reached = {(*case, (r.rows, r.columns), r.wide, r.stream)
               for (case, _), r in zip(asked, routes([line for _, line in asked])) if r.rows and not r.tuned}
    want = set()
    for t, out in RING_TYPES:
        for tile in _ring_tiles(t):
            large = tile[0] * tile[1] > 128 * 128
            want |= {(t, out, form, tile, 1, s) for form in LAYOUT for s in ((0, 1) if large else (0,))}
            if t != "f32" or tile == (64, 64):
                want.add((t, out, c3.FORM_ABT, tile, 0, 0))
    assert not want - reached, sorted(want - reached)


# Results stored element by element: the ring takes 1.1 to 2.6 times as long as the kernel through registers on the first of each
# pair, and less on the second, which has a longer contraction.
@pytest.mark.parametrize("dtype,out,batch,m,n,k,longer", [
    (c3.BF16, c3.BF16, 1, 1067, 5893, 40, 8192), (c3.BF16, c3.F32, 1, 4001, 1041, 784, 8208), (c3.FP8_E4M3, c3.BF16, 8, 4175, 35, 384, 4096),
    (c3.FP8_E4M3, c3.F32, 64, 65, 2057, 80, 8192), (c3.BF16, c3.F32, 1, 1000, 333, 256, 1024)])
def test_odd_results_of_short_contractions_stay_off_the_ring(routes, dtype, out, batch, m, n, k, longer):
    short, long = routes([plain(dtype, c3.FORM_ABT, m, n, x, batch, out) for x in (k, longer)])
    assert not short.rows and long.rows and not short.wide and not long.wide
    for f32_out in (c3.F32, c3.BF16):       # fp32 operands: tiles of 64
        assert [(r.rows, r.columns) for r in routes([plain(c3.F32, c3.FORM_ABT, 3001, 2001, x, out=f32_out) for x in (512, 4096)])] == [(64, 64)] * 2


# Tile-aligned products with few tiles: on the ring where it is clearly faster (9.9 against 14.2 us, 9.9 against 12.5), with the
# tuned kernel where that is (7.5 against 10.1, 10.3 against 12.3, 8.6 against 10.3), the shortest ones too.
@pytest.mark.parametrize("dtype,form,batch,m,n,k,tuned", [
    (c3.BF16, c3.FORM_ABT, 1, 2048, 512, 2048, False), (c3.BF16, c3.FORM_ATB, 1, 512, 2048, 2048, False),
    (c3.BF16, c3.FORM_AB, 1, 2048, 2048, 512, True), (c3.FP8_E4M3, c3.FORM_ATB, 1, 640, 1024, 3840, True),
    (c3.FP8_E4M3, c3.FORM_ABT, 8, 256, 512, 2816, True), (c3.BF16, c3.FORM_AB, 1, 128, 128, 128, True)])
def test_few_aligned_tiles(routes, dtype, form, batch, m, n, k, tuned):
    assert [r.tuned > 0 for r in routes([plain(dtype, form, m, n, k, batch)])] == [tuned]


# The sizes at which the bits of fp8 products are compared between tiles.
def test_compared_fp8_products_run_on_different_tiles(routes):
    tiles = lambda rows: {(f, (r.rows, r.columns)) for f in LAYOUT for r in
                          routes([plain(c3.FP8_E4M3, f, rows or m, n, k) for m, n, k in ps.RING_DEEP]) if not r.tuned}
    assert tiles(0) == {(f, t) for f in LAYOUT for t in ((128, 128), (128, 256), (256, 128))}
    assert {t for rows in (400, 48) for _, t in tiles(rows)} >= {(32, 32), (64, 64)}


# In place: streaming stores in every layout, elements one by one in dX (an odd number of rows of W) and dW (of columns).
def test_gpu_tests_reach_every_way_of_storing_in_place(routes):
    for name in ("bf16", "fp8_e4m3", "f32"):
        asked = [(op, cube(NAMES[name], op, *sizes, out=c3.F32 if name == "f32" else c3.BF16))
                 for sizes in ps.RING_CUBES + ps.RING_CUBES_LINES + ps.RING_CUBES_ODD for op in range(3)]
        reached = {(op, r.wide, r.stream) for (op, _), r in zip(asked, routes([line for _, line in asked])) if r.rows and not r.tuned}
        want = {(op, 1, 0) for op in range(3)} | {(1, 0, 0)}
        if name == "bf16":
            want |= {(2, 0, 0)} | {(op, 1, 1) for op in range(3)}
        if name == "fp8_e4m3":
            want |= {(0, 1, 1), (2, 1, 1)}
        assert not want - reached, (name, want - reached)


@pytest.mark.parametrize("name", sorted(ps.ONE_GB))
def test_operands_above_1_gb_are_kept_off_the_ring(routes, name):
    cols, most, above = ps.ONE_GB[name]
    forms = (c3.FORM_AB, c3.FORM_ABT) + ((c3.FORM_ATB,) if name != "f32" else ())      # (fp32 with few rows has its own kernel)
    for rows, taken in ((most, True), (above, False)):
        lines = [plain(NAMES[name], form, *((cols, 16, rows) if form == c3.FORM_ATB else (rows, 16, cols)), out=c3.F32) for form in forms]
        assert [r.rows > 0 for r in routes(lines)] == [taken] * len(forms)


@pytest.mark.parametrize("name,dtype", [("f32", c3.F32), ("bf16", c3.BF16), ("fp8_e4m3", c3.FP8_E4M3)])
def test_operands_of_4_gb_are_left_to_64_bit_addresses(plans, name, dtype):
    cols, below, above = ps.FOUR_GB[name]
    for rows, taken in ((below, True), (above, False)):
        lines = [plain(dtype, c3.FORM_AB, rows, 16, cols), plain(dtype, c3.FORM_ABT, rows, 16, cols),
                 plain(dtype, c3.FORM_ATB, cols, 16, rows), cube(dtype, 0, 2, rows, cols, 16), cube(dtype, 2, 2, rows, cols, 16)]
        assert [plan[0] > 0 for plan in plans(lines)] == [taken] * 5
