"""GPU parity of the three matrix-product forms on the cube (Algorithms 1-6) against the oracle.

Every step runs through the C ABI on the device: scatter the full operands into their
placements, all-gather, batched local product, reduce-scatter, assemble.  Compared with the
oracle's ``dist3d`` piece by piece (the layouts, bit for bit) and with the plain product of
the full matrices (bit for bit on integers in [-4, 4]; within the stated tolerance on real data).
"""
import numpy as np
import pytest
import torch

import paper_2105_14450_amd as c3
from oracle import dist3d as d3
from oracle import numfmt
from paper_2105_14450_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

AX = {"x": c3.AXIS_X, "y": c3.AXIS_Y, "z": c3.AXIS_Z}
FORM = {"AB": c3.FORM_AB, "ABT": c3.FORM_ABT, "ATB": c3.FORM_ATB}


def _matrix(q, shape, pl, dtype):
    return c3.make_matrix(q, shape[0], shape[1], AX[pl.row_axis], AX[pl.col_axis],
                          c3.SPLIT_ROWS if pl.split == "rows" else c3.SPLIT_COLS, gu.CODE[dtype])


def _shapes(form, u, v, w):
    """A, B, C shapes with result [u, v] and contraction w."""
    return {"AB": ((u, w), (w, v), (u, v)), "ABT": ((u, w), (v, w), (u, v)), "ATB": ((w, u), (w, v), (u, v))}[form]


def _operand(shape, dtype, dist, seed, tid, sigma=1.0):
    raw, scale = synth.store(synth.draw(shape, dist, seed, tid, sigma), dtype, dist == "int")
    return raw, scale, numfmt.decode(raw, dtype, scale)


def _pieces_to_device(q, full_raw, pl, shape, dtype):
    """Full matrix -> cube buffer of pieces on the device, checked against the oracle's slicing."""
    m = _matrix(q, shape, pl, dtype)
    full = gu.to_device(full_raw)
    pieces = gu.empty((q ** 3,) + pl.shard_shape(q, *shape), dtype)
    c3.virtual_cube_matrix_scatter(m, full, pieces)
    want = d3.shard(full_raw, q, pl).reshape((q ** 3,) + pl.shard_shape(q, *shape))
    np.testing.assert_array_equal(gu.raw_host(pieces), want)
    back = gu.empty(shape, dtype)
    c3.virtual_cube_matrix_assemble(m, pieces, back)
    np.testing.assert_array_equal(gu.raw_host(back), full_raw)
    return m, pieces


def _matmul_3d(q, form, a_pieces, ma, pa, sa, b_pieces, mb, pb, sb, pc, sc, dtype, scales, out_dtype, shard_dtype):
    """The four steps on the device; returns the cube buffer of result pieces."""
    n = q ** 3
    a_blocks = gu.empty((n, sa[0] // q, sa[1] // q), dtype)
    b_blocks = gu.empty((n, sb[0] // q, sb[1] // q), dtype)
    c3.virtual_cube_matrix_gather(ma, a_pieces, a_blocks)                    # step 1
    c3.virtual_cube_matrix_gather(mb, b_pieces, b_blocks)                    # step 2
    want_a = d3.all_gather(gu.raw_host(a_pieces).reshape((q, q, q) + pa.shard_shape(q, *sa)), q, pa)
    np.testing.assert_array_equal(gu.raw_host(a_blocks), want_a.reshape(gu.raw_host(a_blocks).shape))
    k = (sa[1] if form != "ATB" else sa[0]) // q
    mm = c3.make_matmul(q, FORM[form], sc[0] // q, sc[1] // q, k, gu.CODE[dtype], gu.CODE[out_dtype],
                        scales[0], scales[1])
    partial = gu.empty((n, sc[0] // q, sc[1] // q), out_dtype)
    nws = c3.cube3d_matmul_workspace_bytes(mm)
    ws = torch.empty(max(nws, 16), dtype=torch.uint8, device="cuda") if nws else None
    c3.cube3d_matmul_blocks(mm, a_blocks, b_blocks, partial, ws)             # step 3
    mc = _matrix(q, sc, pc, shard_dtype)
    out = gu.empty((n,) + pc.shard_shape(q, *sc), shard_dtype)
    c3.virtual_cube_matrix_reduce_scatter(mc, gu.CODE[out_dtype], partial, out)   # step 4
    return mc, out


def _matmul_in_place(q, form, a_pieces, ma, b_pieces, mb, pc, sc, scales, shard_dtype):
    """The same product as one call over the whole cube, pieces read and written in place."""
    mc = _matrix(q, sc, pc, shard_dtype)
    out = gu.empty((q ** 3,) + pc.shard_shape(q, *sc), shard_dtype)
    c3.virtual_cube_matmul(FORM[form], ma, mb, mc, a_pieces, b_pieces, out, scales[0], scales[1])
    return mc, out


def _assemble(mc, pieces, shape, dtype):
    full = gu.empty(shape, dtype)
    c3.virtual_cube_matrix_assemble(mc, pieces, full)
    torch.cuda.synchronize()
    return gu.to_host(full, dtype)


def _compare(got, ref, exact, out_dtype, shard_dtype, tol, what):
    """Integer data: every partial sum is exact in fp32, so with fp32 partials the result is the exact
    product rounded once to the piece dtype: bit for bit.  (bf16 partials round before the sum: within
    tolerance, unless everything is small enough to be exact in bf16 too.)"""
    if exact and out_dtype == "bf16" and np.max(np.abs(ref)) >= 256:
        exact = False
    if exact:
        want = numfmt.round_to_bf16(ref) if shard_dtype == "bf16" else ref
        np.testing.assert_array_equal(got, want, err_msg=what)
    else:
        assert gu.scaled_max_err(got, ref) <= tol, what


CASES = [
    # q, form, result rows, result cols, contraction, dtype, out_dtype, shard_dtype
    (2, "AB", 256, 128, 128, "f32", "f32", "f32"),
    (2, "ABT", 256, 128, 128, "f32", "f32", "f32"),
    (2, "ATB", 256, 128, 128, "f32", "f32", "f32"),
    (3, "ABT", 72, 36, 54, "f32", "f32", "f32"),                  # ragged: the kernels for any size
    (3, "ATB", 36, 72, 45, "bf16", "f32", "bf16"),
    (2, "ABT", 512, 512, 1024, "bf16", "f32", "bf16"),            # tuned kernel, 256-wide blocks
    (2, "ATB", 512, 512, 1024, "bf16", "bf16", "bf16"),
    (2, "AB", 512, 1024, 512, "fp8_e4m3", "f32", "bf16"),
    (2, "ABT", 512, 512, 1024, "fp8_e4m3", "f32", "f32"),
    (4, "ABT", 2048, 2048, 512, "bf16", "f32", "bf16"),           # attention-score-like: 512 x 512 blocks
]


@pytest.mark.parametrize("q,form,u,v,w,dtype,out_dtype,shard_dtype", CASES)
@pytest.mark.parametrize("dist,seed", [("normal", 71), ("int", 171)])
def test_forward_and_backward(q, form, u, v, w, dtype, out_dtype, shard_dtype, dist, seed):
    exact = dist == "int"
    sa, sb, sc = _shapes(form, u, v, w)
    pa, pb, pc = d3.PAPER[form]
    A_raw, a_scale, A = _operand(sa, dtype, dist, seed, synth.TID_X)
    B_raw, b_scale, B = _operand(sb, dtype, dist, seed, synth.TID_W, 0.02 if dist == "normal" else 1.0)
    G_raw, g_scale, G = _operand(sc, dtype, dist, seed, synth.TID_DY)
    ma, a_pieces = _pieces_to_device(q, A_raw, pa, sa, dtype)
    mb, b_pieces = _pieces_to_device(q, B_raw, pb, sb, dtype)
    mg, g_pieces = _pieces_to_device(q, G_raw, pc, sc, dtype)
    tol = gu.TOL[dtype] if shard_dtype == "f32" and out_dtype == "f32" else 2e-2

    # forward: Algorithm 1 / 3 / 5
    mc, c_pieces = _matmul_3d(q, form, a_pieces, ma, pa, sa, b_pieces, mb, pb, sb, pc, sc, dtype,
                              (a_scale, b_scale), out_dtype, shard_dtype)
    C = _assemble(mc, c_pieces, sc, shard_dtype)
    ref = d3.unshard(d3.forward(form, A, B, q), q, pc, *sc)
    _compare(C, ref, exact, out_dtype, shard_dtype, tol, "%s forward" % form)
    mc2, c2 = _matmul_in_place(q, form, a_pieces, ma, b_pieces, mb, pc, sc, (a_scale, b_scale), shard_dtype)
    _compare(_assemble(mc2, c2, sc, shard_dtype), ref, exact, "f32", shard_dtype, tol, "%s forward, in place" % form)
    if exact and out_dtype == "f32":   # same exact sums, same single rounding: the two paths agree bit for bit
        np.testing.assert_array_equal(gu.raw_host(c2), gu.raw_host(c_pieces))

    # backward: Algorithm 2 / 4 / 6, each line one more 3-D product with the placements as stored
    da_ref, db_ref = d3.backward(form, G, A, B, q)
    lines = {"AB": (("ABT", g_pieces, mg, pc, sc, g_scale, b_pieces, mb, pb, sb, b_scale, pa, sa),
                    ("ATB", a_pieces, ma, pa, sa, a_scale, g_pieces, mg, pc, sc, g_scale, pb, sb)),
             "ABT": (("AB", g_pieces, mg, pc, sc, g_scale, b_pieces, mb, pb, sb, b_scale, pa, sa),
                     ("ATB", g_pieces, mg, pc, sc, g_scale, a_pieces, ma, pa, sa, a_scale, pb, sb)),
             "ATB": (("ABT", b_pieces, mb, pb, sb, b_scale, g_pieces, mg, pc, sc, g_scale, pa, sa),
                     ("AB", a_pieces, ma, pa, sa, a_scale, g_pieces, mg, pc, sc, g_scale, pb, sb))}[form]
    for (f2, p1, m1, pl1, s1, sc1, p2, m2, pl2, s2, sc2, plo, so), ref_sh, name in zip(lines, (da_ref, db_ref), "AB"):
        d3.check_directions(f2, pl1, pl2, plo)
        mo, out = _matmul_3d(q, f2, p1, m1, pl1, s1, p2, m2, pl2, s2, plo, so, dtype, (sc1, sc2), out_dtype, shard_dtype)
        got = _assemble(mo, out, so, shard_dtype)
        ref = d3.unshard(ref_sh, q, plo, *so)
        _compare(got, ref, exact, out_dtype, shard_dtype, tol, "%s backward d%s" % (form, name))
        mo2, out2 = _matmul_in_place(q, f2, p1, m1, p2, m2, plo, so, (sc1, sc2), shard_dtype)
        _compare(_assemble(mo2, out2, so, shard_dtype), ref, exact, "f32", shard_dtype, tol,
                 "%s backward d%s, in place" % (form, name))


@pytest.mark.parametrize("q", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8_e4m3"])
def test_every_placement_moves_bits_like_the_oracle(q, dtype):
    rng = np.random.default_rng(5)
    for ra in d3.AXES:
        for ca in d3.AXES:
            if ra == ca:
                continue
            for split in ("rows", "cols"):
                pl = d3.Placement(ra, ca, split)
                shape = (2 * q * q * 4, 3 * q * q * 4)
                raw = rng.integers(0, 120, size=shape).astype(synth.NUMPY_STORAGE[dtype]) if dtype != "f32" else \
                    rng.standard_normal(shape).astype(np.float32)
                m, pieces = _pieces_to_device(q, raw, pl, shape, dtype)
                blocks = gu.empty((q ** 3, shape[0] // q, shape[1] // q), dtype)
                c3.virtual_cube_matrix_gather(m, pieces, blocks)
                want = d3.all_gather(d3.shard(raw, q, pl), q, pl)
                np.testing.assert_array_equal(gu.raw_host(blocks), want.reshape(gu.raw_host(blocks).shape))
                if dtype == "fp8_e4m3":
                    continue
                # reduce-scatter of integer-valued partial blocks: exact sums, piece s kept by processor s
                vals = rng.integers(-4, 5, size=(q, q, q, shape[0] // q, shape[1] // q)).astype(np.float32)
                part_raw, _ = synth.store(vals.reshape(q ** 3, shape[0] // q, shape[1] // q), dtype, True)
                out = gu.empty((q ** 3,) + pl.shard_shape(q, *shape), "f32")
                mo = _matrix(q, shape, pl, "f32")
                c3.virtual_cube_matrix_reduce_scatter(mo, gu.CODE[dtype], gu.to_device(part_raw), out)
                ref = d3.reduce_scatter(vals.astype(np.float64), q, pl)
                np.testing.assert_array_equal(gu.to_host(out, "f32"), ref.reshape(gu.to_host(out, "f32").shape))


def test_shape_sweep_many_items_per_workgroup():
    """Larger single problems whose tile counts exceed the chip's resident workgroups by odd factors
    (persistent workgroups with unequal item counts, tile grids that are no multiple of 8), every
    element against the oracle's exact sums on integer data."""
    _sweep(12, [2304, 2560, 2816, 3072, 3328, 4352], [256, 512, 1024], [1], 500, seed=77)


def test_shape_sweep_of_the_batched_product():
    """Many tile-aligned and ragged block shapes through cube3d_matmul_blocks (q = 1: one problem,
    q = 2: eight problems per launch), all three forms, bf16 and fp8, fp32 and bf16 results: every
    tile size, K-tile depth, split and work-item count the plan can choose.  Integer data: every
    entry must equal the oracle's exact sum (rounded once when the result is bf16)."""
    _sweep(60, [128, 256, 384, 512, 640, 768, 1024, 1280, 1536, 200, 72], [128, 256, 384, 512, 1024, 2048, 4096, 96],
           [1, 1, 2], 300, seed=2024)


def _sweep(trials, sizes, ks, qs, seed0, seed):
    from oracle import matmul as om
    rng = np.random.default_rng(seed)
    done = 0
    for trial in range(trials):
        q = int(rng.choice(qs))
        m, n, k = int(rng.choice(sizes)), int(rng.choice(sizes)), int(rng.choice(ks))
        form = str(rng.choice(["AB", "ABT", "ATB"]))
        dtype = str(rng.choice(["bf16", "bf16", "fp8_e4m3"]))
        out_dtype = str(rng.choice(["f32", "bf16"]))
        nb = q ** 3
        sa, sb, _ = _shapes(form, m, n, k)
        a_raw, _ = synth.store(synth.draw((nb,) + sa, "int", seed0 + trial, synth.TID_X), dtype, True)
        b_raw, _ = synth.store(synth.draw((nb,) + sb, "int", seed0 + trial, synth.TID_W), dtype, True)
        mm = c3.make_matmul(q, FORM[form], m, n, k, gu.CODE[dtype], gu.CODE[out_dtype])
        out = gu.empty((nb, m, n), out_dtype)
        nws = c3.cube3d_matmul_workspace_bytes(mm)
        ws = torch.empty(max(nws, 16), dtype=torch.uint8, device="cuda") if nws else None
        print("sweep %d: q=%d %s m=%d n=%d k=%d %s -> %s ws=%d" % (trial, q, form, m, n, k, dtype, out_dtype, nws), flush=True)
        c3.cube3d_matmul_blocks(mm, gu.to_device(a_raw), gu.to_device(b_raw), out, ws)
        torch.cuda.synchronize()
        got = gu.to_host(out, out_dtype)
        threads = min(16, om.max_threads())
        for r in range(nb):     # every element of every processor's block
            A, B = numfmt.decode(a_raw[r], dtype), numfmt.decode(b_raw[r], dtype)
            fn = {"AB": om.forward, "ABT": om.backward_dx, "ATB": om.backward_dw}[form]
            ref = fn(A, B, threads)
            want = numfmt.round_to_bf16(ref) if out_dtype == "bf16" else ref
            np.testing.assert_array_equal(got[r], want, err_msg="trial %d block %d" % (trial, r))
        done += 1
    assert done == trials
