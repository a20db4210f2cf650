// Dispatch of the product kernel for any size (gemm_edge.h).
#include "gemm_edge.h"

namespace cube3d {
using namespace edge;

namespace {

constexpr int64_t MAX_EXTENT = (1ll << 31) - 4096;   // indices stay below 2^31, also those of the K-tiles in flight at the end

// widest power of two up to 16 / es elements that divides `x`
int64_t common_piece(int64_t piece, int64_t x)
{
    while (x & (piece - 1)) piece /= 2;
    return piece;
}

// An index that is not cut into shards: one panel longer than any extent.
AxisMap plain_map(int64_t u)
{
    return AxisMap{INT32_MAX, INT32_MAX, 0, 0, u};
}

// Largest element offset of an operand or of the output (offsets grow with the panel, shard and element numbers).
int64_t last_offset(const AxisMap &m, int64_t extent)
{
    const int64_t blocks = (extent - 1) / m.P1, in_block = blocks ? m.P1 - 1 : extent - 1;
    const int64_t shards = in_block / m.P2, in_shard = shards ? m.P2 - 1 : in_block;
    return blocks * m.s1 + shards * m.s2 + in_shard * m.u;
}

// elements that can be read at once along the contiguous index `c` of an operand whose other index is `r`
int64_t piece_of(const AxisMap &c, const AxisMap &r, int64_t extent, int64_t batch_stride, int64_t widest)
{
    if (c.u != 1) return 1;
    int64_t piece = common_piece(widest, extent);
    if (c.P2 != INT32_MAX) piece = common_piece(piece, c.P2);
    for (int64_t x : {c.s1, c.s2, r.s1, r.s2, r.u, batch_stride}) piece = common_piece(piece, x);
    return piece;
}

// Estimated time of a launch in us, to compare this kernel with the element-wise one (gemm_generic) where the
// contraction is short: a workgroup here pays for its pipeline's start and its staged output however few K-tiles it
// has, an element-wise one next to nothing besides its steps of 32.  Fitted to products of 1-4096 blocks on one
// MI355X, all kernels timed at each.  Over 3130 products the choice is 1.1 % slower than the best one in the mean, and at
// 56 of them more than 5 % slower than the element-wise kernel (at most 1.44 times; with the tile rule alone at 1400,
// up to 8 times).
//   start: launch, first loads, output;  tile, ktile, full: per workgroup, per K-tile of it, and more per K-tile the fuller
//   the tiles are, when all CUs are busy
// (These are the kernel through registers: where the ring kernel would take the product, its time is not asked.)
struct Cost {
    float start, tile, ktile, full;
};
constexpr Cost COST[8][3] = {
    // tiles of 32                       64                                  128
    {{5.14f, 0.48f, 0.05f, 0.09f}, {5.46f, 1.14f, 0.24f, 0.19f}, {7.30f, 2.48f, 0.00f, 1.01f}},    // bf16, loads of 16 bytes
    {{5.79f, 0.62f, 0.13f, 0.28f}, {7.56f, 0.96f, 0.39f, 0.39f}, {8.90f, 4.92f, 0.00f, 2.17f}},    //       4
    {{6.02f, 0.84f, 0.27f, 0.60f}, {7.88f, 1.35f, 0.65f, 0.93f}, {12.4f, 3.97f, 0.28f, 3.93f}},    //       2
    {{5.21f, 0.49f, 0.04f, 0.10f}, {5.46f, 1.25f, 0.00f, 0.41f}, {6.87f, 2.42f, 0.00f, 1.34f}},    // fp8, loads of 16 bytes
    {{5.86f, 0.63f, 0.13f, 0.18f}, {7.27f, 1.08f, 0.16f, 0.88f}, {10.2f, 4.56f, 0.00f, 2.37f}},    //      4
    {{6.61f, 1.28f, 0.76f, 0.97f}, {8.12f, 2.67f, 1.52f, 1.89f}, {}},                              //      1 (no tiles of 128)
    {{5.32f, 0.85f, 0.17f, 0.07f}, {6.02f, 1.32f, 0.53f, 0.31f}, {7.87f, 3.79f, 0.85f, 1.88f}},    // fp32, loads of 16 bytes
    {{5.38f, 0.90f, 0.20f, 0.22f}, {7.61f, 1.18f, 0.56f, 0.60f}, {12.4f, 5.25f, 0.73f, 2.83f}},    //       4
};
//   step, full: per workgroup and step of 32, and more of it the fuller the tiles are (elements beyond the edges are not loaded)
//   least: workgroups per CU below which a step gets no faster, for one block or about one workgroup per CU;  several:
//   for more blocks, which share less through the caches;  one: what a step of one block's workgroups takes of that
struct ElementCost {
    float start, least, several, step, full, one;
};
constexpr ElementCost ELEMENT_COST[3] = {{4.73f, 2.26f, 3.47f, 0.40f, 0.64f, 0.94f},      // bf16
                                         {4.65f, 2.41f, 3.64f, 0.38f, 0.53f, 0.91f},      // fp8
                                         {4.34f, 1.70f, 3.23f, 0.80f, 0.84f, 0.90f}};     // fp32
constexpr float ELEMENT_MAPS = 3.f;      // an index map divides four times per element: 2.4-3.2 times a step's time
// Beyond, its steps leave the caches and the fit: sooner with several blocks on few workgroups per CU (8 of 407 x 521 x 799
// fp8 in single bytes 60 here against 121 us), later with single bytes and mostly full tiles (3001 x 3001 x 1025 286
// against 253, x 2049 523 against 506; but 4096 blocks of 41 x 41 x 1025 397 against 433).
constexpr int64_t SHORT_FEW = 384, SHORT = 640, SHORT_SINGLE_BYTES = 2048;

bool element_wise_is_faster(const GemmArgs &g, int tile, int piece, int64_t workgroups, int64_t workgroups64)
{
    const int type = g.in_dtype == CUBE3D_BF16 ? 0 : g.in_dtype == CUBE3D_FP8_E4M3 ? 1 : 2;
    const int es = type == 0 ? 2 : type == 1 ? 1 : 4, width = piece >= 16 ? 0 : piece >= 4 ? 1 : 2;
    const double elements = (double)g.Mo * (double)g.No * g.batch;
    const float cus = (float)num_compute_units(), per_cu = (float)workgroups / cus, per_cu64 = (float)workgroups64 / cus;
    const float full = (float)(elements / ((double)workgroups * tile * tile));
    const float full64 = (float)(elements / ((double)workgroups64 * 64 * 64));
    const bool one = g.batch == 1, single_bytes = es == 1 && width == 2;
    const int64_t limit = !one && per_cu64 < 6.f ? SHORT_FEW : single_bytes && full64 >= 0.5f ? SHORT_SINGLE_BYTES : SHORT;
    if (g.Kc > limit) return false;
    const Cost &c = COST[3 * type + width][tile == 32 ? 0 : tile == 64 ? 1 : 2];
    const float ktiles = (float)((g.Kc * es + BKB - 1) / BKB);
    const float here = c.start + (per_cu > 1.f ? per_cu : 1.f) * (c.tile + (c.ktile + c.full * full) * ktiles);
    const ElementCost &e = ELEMENT_COST[type];
    const float least = one || per_cu64 <= 1.3f ? e.least : e.several, busy = one ? e.one * per_cu64 : per_cu64;
    const float steps = (float)((g.Kc + 31) / 32) * (g.maps ? ELEMENT_MAPS : 1.f);
    return e.start + steps * (busy > least ? busy : least) * (e.step + e.full * full64) < here;
}

// A launch has fewer than 2^32 work-items along a grid dimension: 2^24 workgroups of 256.
constexpr int64_t MAX_WORKGROUPS = (1ll << 24) - 1;

}  // namespace

namespace edge {

int make_plan(const GemmArgs &g, Plan *plan)
{
    const int es = g.in_dtype == CUBE3D_F32 ? 4 : g.in_dtype == CUBE3D_BF16 ? 2 : g.in_dtype == CUBE3D_FP8_E4M3 ? 1 : 0;
    if (es == 0 || (g.out_dtype != CUBE3D_F32 && g.out_dtype != CUBE3D_BF16)) return CUBE3D_ENOTIMPL;
    if (g.Mo < 1 || g.No < 1 || g.Kc < 1 || g.batch < 1 || (!g.a_kmajor && g.b_kmajor)) return CUBE3D_ENOTIMPL;
    if (g.Mo > MAX_EXTENT || g.No > MAX_EXTENT || g.Kc > MAX_EXTENT) return CUBE3D_ENOTIMPL;
    if (g.maps && g.batch != 1) return CUBE3D_ENOTIMPL;
    if ((g.Mo + 63) / 64 > 65535 || g.batch > 65535) return CUBE3D_ENOTIMPL;   // refused by gemm_generic
    Params &p = plan->params;
    p = Params{};
    if (g.maps) {
        p.maps = *g.maps;
    } else {
        p.maps.a_mn = plain_map(g.a_kmajor ? g.lda : 1);
        p.maps.a_k = plain_map(g.a_kmajor ? 1 : g.lda);
        p.maps.b_mn = plain_map(g.b_kmajor ? g.ldb : 1);
        p.maps.b_k = plain_map(g.b_kmajor ? 1 : g.ldb);
        p.maps.c_m = plain_map(g.ldc);
        p.maps.c_n = p.maps.bias_n = plain_map(1);
        p.sA = g.strideA * es;
        p.sB = g.strideB * es;
    }
    GemmMaps &m = p.maps;
    for (AxisMap *x : {&m.a_mn, &m.a_k, &m.b_mn, &m.b_k, &m.c_m, &m.c_n, &m.bias_n}) {
        if (x->P1 < 1 || x->P2 < 1 || x->P1 % x->P2) return CUBE3D_ENOTIMPL;
        prepare_axis_map(*x);
    }
    // an operand element is buffer start + 32-bit byte offset
    if ((last_offset(m.a_mn, g.Mo) + last_offset(m.a_k, g.Kc) + 1) * es >= (1ll << 32)) return CUBE3D_ENOTIMPL;
    if ((last_offset(m.b_mn, g.No) + last_offset(m.b_k, g.Kc) + 1) * es >= (1ll << 32)) return CUBE3D_ENOTIMPL;
    const int64_t widest = 16 / es;
    const int64_t pa = g.a_kmajor ? piece_of(m.a_k, m.a_mn, g.Kc, g.maps ? 0 : g.strideA, widest)
                                  : piece_of(m.a_mn, m.a_k, g.Mo, g.maps ? 0 : g.strideA, widest);
    const int64_t pb = g.b_kmajor ? piece_of(m.b_k, m.b_mn, g.Kc, g.maps ? 0 : g.strideB, widest)
                                  : piece_of(m.b_mn, m.b_k, g.No, g.maps ? 0 : g.strideB, widest);
    const int piece = plan->piece = (int)(pa < pb ? pa : pb) * es;
    const int oes = g.out_dtype == CUBE3D_F32 ? 4 : 2;
    p.sC = g.maps ? 0 : g.strideC * oes;
    p.out_f32 = oes == 4;
    p.out_wide = piece_of(m.c_n, m.c_m, g.No, g.maps ? 0 : g.strideC, 16 / oes) * oes == 16;
    p.A = static_cast<const char *>(g.A);
    p.B = static_cast<const char *>(g.B);
    p.C = static_cast<char *>(g.C);
    p.Mo = (int)g.Mo; p.No = (int)g.No; p.Kc = (int)g.Kc;
    p.alpha = g.alpha;
    p.step_a = (unsigned)(BKB * m.a_k.u);
    p.step_b = (unsigned)(BKB * m.b_k.u);
    auto tiles = [&](int64_t t) { return ((g.Mo + t - 1) / t) * ((g.No + t - 1) / t) * g.batch; };
    // Tile side: the largest that still gives most CUs a tile, because a CU without one costs more than the
    // smaller tile's extra LDS reads.  bf16, us with 128 / 64 / 32 at (Mo, No, Kc): (2997, 1152, 4608) with B K-major = 216 tiles
    // of 128: 52 / 66 / 93; (3000, 1024, 4096) = 192: 46 / 47 / 70; (1000, 2048, 1024) = 128, fp8: 15 / 11 / 14;
    // (384, 1536, 999) with no operand K-major = 144 tiles of 64: 18 / 10.7 / 12.7; (64, 8192, 2048) = 128: 27 / 15.7 / 15.3;
    // (999, 384, 1536) = 96: 22 / 12.7 / 10.8; (64, 2048, 8192) = 32: 84 / 40 / 24.  The other types and widths cross at the
    // same places: fp32 (1004, 1004, 1028) = 256 tiles of 64: 78 / 33 / 34, (404, 404, 1028) = 49: 76 / 29 / 14; bf16 in
    // single elements (3001, 3001, 1025) = 576 of 128: 182 / 207 / 532, (1001, 1001, 1025) = 256 of 64: 67 / 30 / 60,
    // (401, 401, 1025) = 49: 67 / 30 / 20.  Not so fp32 (3004, 3004, 1028), 576 tiles of 128 for 512 places: 213 / 187 / 216.
    // And not where most of the larger tile lies beyond the output: it takes the time of two to three half as wide.
    // 4096 blocks, bf16: 41 x 41 x 1025 684 / 370 / 662, 41 x 41 x 129 151 / 70 / 130, 9 x 9 x 1025 481 / 222 / 120,
    // 24 x 104 x 1032 224 / 250 / 304; 512 of 101 x 201 x 257 82 / 122 / 220; fp8, 304 x 528 x 144 121 / 162 / 253.
    const int64_t cus = num_compute_units(), t32 = tiles(32), t64 = tiles(64), t128 = tiles(128);
    const bool single_bytes = piece < 4 && es == 1;      // no 128 x 128 kernel, see launch_tile
    const bool large = t128 > cus * 3 / 4 && 2 * t64 >= 5 * t128 && !single_bytes, medium = t64 > cus / 2 && t32 >= 2 * t64;
    const int tile = plan->tile = large ? 128 : medium ? 64 : 32;
    if (element_wise_is_faster(g, tile, piece, tiles(tile), t64)) return CUBE3D_ENOTIMPL;
    if (tiles(tile) > MAX_WORKGROUPS) return CUBE3D_ENOTIMPL;
    p.tiles_m = (int)((g.Mo + tile - 1) / tile);
    p.tiles_n = (int)((g.No + tile - 1) / tile);
    p.group_m = 8;
    return CUBE3D_OK;
}

}  // namespace edge

namespace {

// Time of a ring launch in us: start, then per round of workgroups item (more with fp32 results) and ktile per K-tile;
// pair: two workgroups on a CU (tiles of 32 and 64); the same with both operands K-major.  Fitted to 810 products of 8-8192
// rows, 128-8192 columns, 35-8192 indices and 1-64 blocks on one MI355X, all tiles timed at each: the choice takes 0.6-1.4 %
// longer than the best tile in the mean, and less than 0.80 of the time without the ring kernel (fp32 0.94).  15208 others whose
// sizes are multiples of 16 bytes: 0.83 of the time without it, 49 over 4 % longer, at most 1.15 times.
struct RingCost {
    int tile_m, tile_n;
    float start, item, wide, ktile, pair, ktile_kk, pair_kk;
};
constexpr RingCost RING_BF16[] = {{32, 32, 3.67f, 0.52f, 0.06f, 0.166f, 0.485f, 0.146f, 0.335f},
                                  {64, 64, 3.69f, 0.80f, 0.27f, 0.165f, 0.389f, 0.150f, 0.370f},
                                  {128, 128, 2.65f, 3.15f, 1.26f, 0.374f, 0.f, 0.333f, 0.f},
                                  {128, 256, 2.34f, 5.30f, 2.37f, 0.558f, 0.f, 0.519f, 0.f},
                                  {256, 128, 2.59f, 4.97f, 2.41f, 0.560f, 0.f, 0.510f, 0.f}};
constexpr RingCost RING_FP8[] = {{32, 32, 3.76f, 0.47f, 0.00f, 0.234f, 0.736f, 0.213f, 0.427f},       // bf16 results
                                 {64, 64, 3.75f, 0.84f, 0.00f, 0.224f, 0.532f, 0.251f, 0.495f},
                                 {128, 128, 2.95f, 2.91f, 0.00f, 0.396f, 0.f, 0.345f, 0.f},
                                 {128, 256, 2.71f, 4.93f, 0.00f, 0.528f, 0.f, 0.523f, 0.f},
                                 {256, 128, 2.90f, 4.69f, 0.00f, 0.548f, 0.f, 0.526f, 0.f}};
constexpr RingCost RING_FP8_F32[] = {{32, 32, 3.82f, 0.47f, 0.00f, 0.234f, 0.675f, 0.208f, 0.459f},   // fp32 results
                                     {64, 64, 3.66f, 1.11f, 0.00f, 0.235f, 0.488f, 0.244f, 0.532f},
                                     {128, 128, 2.58f, 4.20f, 0.00f, 0.548f, 0.f, 0.559f, 0.f},
                                     {128, 256, 3.00f, 6.40f, 0.00f, 0.999f, 0.f, 0.989f, 0.f},
                                     {256, 128, 3.18f, 6.12f, 0.00f, 0.981f, 0.f, 0.893f, 0.f}};
constexpr RingCost RING_F32[] = {{64, 64, 3.63f, 1.40f, 0.00f, 0.535f, 1.016f, 0.508f, 0.925f},
                                 {128, 128, 2.52f, 5.02f, 0.00f, 1.801f, 0.f, 1.801f, 0.f}};
constexpr float PAIR_ITEM = 1.7f;      // an item's fixed part with two workgroups on the CU

// What the ring kernel assumes of an operand: offsets below its buffer's size, the k-rows of a K-tile within half of that, and
// shards of the contraction index that are whole and no shorter than a K-tile.  The longest K-tile that fits, in indices.
int64_t longest_ring_ktile(const AxisMap &mn, const AxisMap &k, bool kmajor, int64_t extent, int64_t Kc, int es)
{
    if ((last_offset(mn, extent) + last_offset(k, Kc) + 1) * es > (int64_t)RING_SPAN) return 0;
    int64_t longest = kmajor ? INT32_MAX : (int64_t)RING_SPAN / 2 / (k.u * es);
    if (k.P2 != INT32_MAX) longest = Kc % k.P2 ? 0 : longest < k.P2 ? longest : k.P2;
    return longest;
}

// Results that are stored element by element (output rows that are not whole 16-byte pieces) cost a tile of the ring kernel more
// than one of the kernel through registers: bytes of contraction from which the ring makes up for that.  Ring against
// registers, A B^T of an odd number of columns: tiles of 256 x 128 took 1.5 times as long at 512 bytes (bf16), 1.2 at 4096 and 0.9 at
// 16384; tiles of 64 with fp32 results 1.03 at 512, 0.98 at 1024.  Of 14149 products 3986 took over 4 % longer on the ring, with
// these lines 227.  (fp32 operands: no tiles of 128 for such results, 1.08-1.23 at every length; 0.87 in tiles of 64.)
int64_t least_narrow_bytes(const RingPlan &r, bool f32, bool fp8, bool wide_results)
{
    const int area = r.tile_m * r.tile_n;
    if (area <= 32 * 32) return 768;
    if (area <= 64 * 64) return wide_results && !f32 ? 1024 : 256;
    if (fp8 && !wide_results) return 4096;
    return area == 128 * 128 && !fp8 ? 12288 : 8192;
}

}  // namespace

namespace edge {

RingPlan ring_plan(const GemmArgs &g, const Plan &plan)
{
    RingPlan best{0, 0, 0.f};
    const bool f32 = g.in_dtype == CUBE3D_F32, fp8 = g.in_dtype == CUBE3D_FP8_E4M3;
    const int es = f32 ? 4 : fp8 ? 1 : 2;
    if (plan.piece < 16) return best;
    if (plan.params.maps.bias && (!g.a_kmajor || g.b_kmajor)) return best;     // the ring adds a bias in the forward layout only
    // Few rows in fp32: the wavefronts of a 32 x 32 tile share its k-steps, a quarter of the chain (10 x 384 x 3904: 28 us, 69 on
    // the ring's tiles of 64).  One K-tile of 256 bytes: nothing to keep in flight (85 x 448 x 128 fp8 4.5 against 4.7 us).
    if (plan.tile == 32 && (f32 || g.Kc * es <= 256)) return best;
    const bool wide = g.out_dtype == CUBE3D_F32, kk = g.a_kmajor && g.b_kmajor;
    const RingCost *costs = f32 ? RING_F32 : fp8 ? (wide ? RING_FP8_F32 : RING_FP8) : RING_BF16;
    const int n = f32 ? 2 : 5;
    const int64_t cus = num_compute_units();
    const GemmMaps &m = plan.params.maps;
    const int64_t longest_a = longest_ring_ktile(m.a_mn, m.a_k, g.a_kmajor, g.Mo, g.Kc, es);
    const int64_t longest_b = longest_ring_ktile(m.b_mn, m.b_k, g.b_kmajor, g.No, g.Kc, es);
    for (int i = 0; i < n; ++i) {
        const RingCost &c = costs[i];
        const int kb = ring_ktile_bytes(c.tile_n);
        if (kb / es > longest_a || kb / es > longest_b) continue;
        if (f32 && !plan.params.out_wide && c.tile_m > 64) continue;      // (least_narrow_bytes)
        const int64_t items = ((g.Mo + c.tile_m - 1) / c.tile_m) * ((g.No + c.tile_n - 1) / c.tile_n) * g.batch;
        const bool pair = c.pair > 0.f && items > cus;
        const float rounds = (float)((items + (pair ? 2 : 1) * cus - 1) / ((pair ? 2 : 1) * cus)), ktiles = (float)((g.Kc * es + kb - 1) / kb);
        const float item = (c.item + (wide ? c.wide : 0.f)) * (pair ? PAIR_ITEM : 1.f);
        const float ktime = pair ? (kk ? c.pair_kk : c.pair) : (kk ? c.ktile_kk : c.ktile);
        const float us = c.start + rounds * (item + ktiles * ktime);
        if (best.tile_m == 0 || us < best.us) best = RingPlan{c.tile_m, c.tile_n, us};
    }
    if (best.tile_m > 0 && !plan.params.out_wide && g.Kc * es < least_narrow_bytes(best, f32, fp8, wide)) return RingPlan{0, 0, 0.f};
    return best;
}

// Results that would take half of the eight 4 MB L2s from the operands' panels are written past them: three fp8 products of
// 3000 x 3072 x 12288 389 -> 363 us, 27 blocks of 1000 x 1536 x 512 63 -> 57.  Smaller ones the next call finds in the caches: an
// fp8 layer whose partial products take 10 MB lost 2 % with streaming stores.  Only whole cache lines, that is where the 128
// bytes that eight lanes of an output row store are one: 64 blocks of 2934 x 1608 x 80 with fp32 results, whose rows end inside
// a line, took 697 us with streaming stores and 405 without.  Tiles above 128 x 128 only: 1-2 % lost with smaller ones.
bool ring_streams(const GemmArgs &g, const Params &p, const RingPlan &r)
{
    const int es = p.out_f32 ? 4 : 2;
    if (r.tile_m * r.tile_n <= 128 * 128 || g.Mo * g.No * g.batch * es <= (16ll << 20)) return false;
    const AxisMap &m = p.maps.c_m, &n = p.maps.c_n;
    for (int64_t x : {m.u, m.s1, m.s2, n.s1, n.s2})
        if (x * es % 128) return false;
    return n.u == 1 && (n.P2 == INT32_MAX || (int64_t)n.P2 * es % 128 == 0) && p.sC % 128 == 0 && (uintptr_t)p.C % 128 == 0;
}

}  // namespace edge

// Both estimates are a few per cent off: of 12167 tile-aligned products with few tiles 822 took over 4 % longer on the ring when
// the lower one decided, with these margins some 130 would.  Between 0.95 and 1 of the tuned kernel's estimate the two are even
// (0.90-1.12 of its time, by type and layout); between 0.9 and 0.95 with bf16 results of bf16 K-major operands (1.04) and of fp8
// ones with an MN-major operand among them (0.95).
bool gemm_edge_takes_less(const GemmArgs &g, double us)
{
    const double margin = g.out_dtype == CUBE3D_BF16 && (g.in_dtype == CUBE3D_BF16) == g.b_kmajor ? 0.9 : 0.95;
    // Start and one tile take the ring 4.2 us: up to here it could save no more than the estimate costs the host (0.2-0.4 us, twice
    // that before a plan was made once per call; a call takes it 3.2).
    constexpr double LEAST = 4.6;
    Plan plan;
    if (us * margin <= LEAST || make_plan(g, &plan) != CUBE3D_OK) return false;
    const RingPlan ring = ring_plan(g, plan);
    return ring.tile_m > 0 && ring.us < us * margin;
}

int gemm_edge(const GemmArgs &g)
{
    Plan plan;
    const int rc = make_plan(g, &plan);
    if (rc != CUBE3D_OK) return rc;
    const RingPlan ring = ring_plan(g, plan);
    if (ring.tile_m > 0) {
        switch (g.in_dtype) {
        case CUBE3D_F32: return gemm_ring_f32(g, plan.params, ring);
        case CUBE3D_BF16: return gemm_ring_bf16(g, plan.params, ring);
        default:
            // The 64-deep MFMAs add in another order than the 16-deep ones of all other kernels for any size: where the
            // result is rounded to bf16 and the matrix cores are what bounds the tile.
            return ring.tile_m >= 128 && g.out_dtype == CUBE3D_BF16 ? gemm_ring_fp8_deep(g, plan.params, ring)
                                                                    : gemm_ring_fp8(g, plan.params, ring);
        }
    }
    switch (g.in_dtype) {
    case CUBE3D_F32: return gemm_edge_f32(g, plan.params, plan.tile, plan.piece);
    case CUBE3D_BF16: return gemm_edge_bf16(g, plan.params, plan.tile, plan.piece);
    default: return gemm_edge_fp8(g, plan.params, plan.tile, plan.piece);
    }
}

}  // namespace cube3d
