// Product kernel without size classes, for gfx950: any Mo, No and Kc, fp32 / bf16 / fp8-e4m3 operands, plain
// leading dimensions or a cube of shards read in place.  It takes what the tile-aligned kernel
// (gemm_mfma_kernel.h) declines: ragged sizes, few rows, fp32.  The local products of Algorithm 1 step 3 and
// Algorithm 2 lines 1-2.  Operands that can be read in 16-byte pieces mostly go to the ring kernel instead
// (gemm_ring.h; ring_plan says which); the figures below are this kernel's.
//
// Work split.  A workgroup of four wavefronts makes a T x T tile: T = 128 or 64 as 2 x 2 sub-tiles in 32x32
// MFMA accumulators, T = 32 as 2 x 2 blocks of 16x16 MFMAs (bf16, fp8) or as one block whose k-steps the wavefronts
// share (fp32), for few rows: many workgroups and no second pass.  K-tiles are 128 bytes of the contraction index per row.
// Operands go through registers into LDS, double-buffered, one barrier per K-tile.  Registers rather than
// direct-to-LDS loads because a piece may be narrower than 16 bytes, may lie in another shard than its
// neighbour, and has to be zero beyond the last contraction index.
//
// What bounds it.  With few workgroups per CU the chain of one K-tile: 64 rows x 8192 x 2048 bf16 took 63 us on 32
// tiles of 64 with one K-tile of loads in flight; four in flight, waits that count exactly one K-tile's loads and
// fragment reads ahead of the LDS writes made it 40, the 32 x 32 tiles and one vector addition per load in place of a
// per-lane walk 24 (33 MB of weights: 5 us at 7 TB/s).  32 x 32 tiles whose wavefronts shared the k-steps, as in
// fp32, took 22 there and 23 against 26 for 64 x 2048 x 8192 with W^T, but 7.2 against 6.7 for 64 x 512 x 512, and
// their four partial sums made a row's bits depend on how many rows the call had.  With many workgroups LDS reads
// and vector instructions share the time with the MFMAs: 6000 x 3000 x 5000 bf16 takes 232-252 us = 0.71-0.78
// PFLOP/s, three fp8 products of 3000 x 3072 x 12288 590 us = 1.15 PFLOP/s; the element-wise kernel makes 30-45
// TFLOP/s at these sizes.
//
// Edges.  Rows and columns beyond the output are read from the last valid one (their sums are never
// stored), so bounds are looked at along the contraction only: a piece beyond its end is read from element 0 and
// written as zeros.  The prologue does that and the loop over the last D + 1 to 2 D + 1 K-tiles (D in flight);
// the loop proper starts with more than 2 D whole K-tiles.  Both operands are read in pieces of GB bytes: 16, 4 or
// one element's, the widest that divides every distance and extent along both contiguous indices, so no piece
// straddles a row, a shard or the buffer's end.
//
// Address arithmetic.  Plain operands are a map with one endless panel.  From one K-tile to the next all of a
// lane's byte offsets grow by one distance; only where a shard ends are they taken from the index map again (with
// multiplications, nothing is divided), so a K-tile costs one vector addition per load.
#pragma once
#include <type_traits>

#include "common.h"

namespace cube3d {
namespace edge {

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int BKB = 128;      // bytes of contraction index per K-tile and row

// Element traits.  M32 and M16 are the matrix instructions on 32 x 32 and 16 x 16 blocks: a step is what one
// LDS fragment covers, KSTEP contraction indices of which the lane groups (lane / SIDE) hold consecutive runs, the same
// for both kinds of operand.  In bf16 and fp8 every output element adds its products in ascending order in one
// accumulator, and M16 gives the bits of M32 (compared on random operands over 512 indices): a row of the
// result does not depend on the tile side, that is on how many other rows the call has.
//   mn_swz: slot permutation of an MN-major row (spr 16-byte slots) in k-row k, so that the k-rows that one
//   read covers lie in different banks (32 x 32 tiles: 26.2 -> 24.4 us for 64 x 8192 x 2048)
struct Bf16 {
    static constexpr int ELT = 2;
    __device__ static __forceinline__ int mn_swz(int k, int spr)
    {
        return spr >= 16 ? 4 * (k & 3) : spr >= 8 ? 4 * ((k >> 1) & 1) : 2 * ((k >> 3) & 1);
    }
    struct M32 {
        static constexpr int SIDE = 32, KSTEP = 16, MFMAS = 1;      // MFMAS: MFMAs per fragment pair
        typedef i32x4 Frag;
        typedef f32x16 Acc;
        // bytes [16 * slot, +16) of a K-major row hold 8 k: slot 2 * step + group is a fragment
        __device__ static __forceinline__ Frag read_k(const char *row, int swz, int step, int g)
        {
            return *reinterpret_cast<const i32x4 *>(row + (((2 * step + g) ^ swz) * 16));
        }
        // transposing reads: 16 lanes take 4 k-rows x 16 columns, lane n receives the 4 k of column n
        template <int RB> __device__ static __forceinline__ Frag read_mn(const char *tile, int lane, int col0, int step)
        {
            const int g = lane / 16;
            return read_mn_at<RB>(tile + step * KSTEP * RB, lane % 16, col0 + 16 * (g % 2), 8 * (g / 2));
        }
        __device__ static __forceinline__ Acc mfma(Frag a, Frag b, Acc c, int)
        {
            return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
        }
    };
    struct M16 {
        static constexpr int SIDE = 16, KSTEP = 32, MFMAS = 1;
        typedef i32x4 Frag;
        typedef f32x4 Acc;
        __device__ static __forceinline__ Frag read_k(const char *row, int swz, int step, int g)
        {
            return *reinterpret_cast<const i32x4 *>(row + (((4 * step + g) ^ swz) * 16));
        }
        template <int RB> __device__ static __forceinline__ Frag read_mn(const char *tile, int lane, int col0, int step)
        {
            return read_mn_at<RB>(tile + step * KSTEP * RB, lane % 16, col0, 8 * (lane / 16));
        }
        __device__ static __forceinline__ Acc mfma(Frag a, Frag b, Acc c, int)
        {
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
        }
    };
    // 8 k from k-row k0 on (a multiple of 8) of 16 columns, for the 16 lanes s of a group
    template <int RB> __device__ static __forceinline__ i32x4 read_mn_at(const char *tile, int s, int col0, int k0)
    {
        const int k = k0 + s / 4, byte = (col0 + 4 * (s % 4)) * 2;
        const char *ad = tile + k * RB + (((byte / 16) ^ mn_swz(k, RB / 16)) * 16) + byte % 16;
        auto rd = [](const char *a) {
            return __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4 *)(__attribute__((address_space(3))) const char *)a));
        };
        const i32x2 lo = rd(ad), hi = rd(ad + 4 * RB);
        return i32x4{lo[0], lo[1], hi[0], hi[1]};
    }
};

struct Fp8 {
    static constexpr int ELT = 1;
    __device__ static __forceinline__ int mn_swz(int k, int spr)
    {
        return spr >= 8 ? 2 * ((k >> 1) & 3) : spr >= 4 ? 2 * ((k >> 2) & 1) : (k >> 3) & 1;
    }
    struct M32 {
        static constexpr int SIDE = 32, KSTEP = 16, MFMAS = 1;
        typedef i32x2 Frag;
        typedef f32x16 Acc;
        __device__ static __forceinline__ Frag read_k(const char *row, int swz, int step, int g)
        {
            return *reinterpret_cast<const i32x2 *>(row + ((step ^ swz) * 16) + 8 * g);
        }
        template <int RB> __device__ static __forceinline__ Frag read_mn(const char *tile, int lane, int col0, int step)
        {
            const int g = lane / 16;
            return read_mn_at<RB>(tile + step * KSTEP * RB, lane % 16, col0 + 16 * (g % 2), 8 * (g / 2));
        }
        __device__ static __forceinline__ Acc mfma(Frag a, Frag b, Acc c, int)
        {
            return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(__builtin_bit_cast(long, a), __builtin_bit_cast(long, b), c, 0, 0, 0);
        }
    };
    struct M16 {
        static constexpr int SIDE = 16, KSTEP = 32, MFMAS = 1;
        typedef i32x2 Frag;
        typedef f32x4 Acc;
        __device__ static __forceinline__ Frag read_k(const char *row, int swz, int step, int g)
        {
            return *reinterpret_cast<const i32x2 *>(row + (((2 * step + g / 2) ^ swz) * 16) + 8 * (g % 2));
        }
        template <int RB> __device__ static __forceinline__ Frag read_mn(const char *tile, int lane, int col0, int step)
        {
            return read_mn_at<RB>(tile + step * KSTEP * RB, lane % 16, col0, 8 * (lane / 16));
        }
        __device__ static __forceinline__ Acc mfma(Frag a, Frag b, Acc c, int)
        {
            return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(__builtin_bit_cast(long, a), __builtin_bit_cast(long, b), c, 0, 0, 0);
        }
    };
    // transposing read: 16 lanes take 8 k-rows x 16 columns, lane n receives the 8 k of column n
    template <int RB> __device__ static __forceinline__ i32x2 read_mn_at(const char *tile, int s, int col0, int k0)
    {
        const int k = k0 + s / 2, byte = col0 + 8 * (s % 2);
        const char *ad = tile + k * RB + (((byte / 16) ^ mn_swz(k, RB / 16)) * 16) + byte % 16;
        return __builtin_amdgcn_ds_read_tr8_b64_v2i32(
            (__attribute__((address_space(3))) i32x2 *)(__attribute__((address_space(3))) const char *)ad);
    }
};

struct F32 {
    static constexpr int ELT = 4;
    __device__ static __forceinline__ int mn_swz(int k, int spr) { return spr >= 16 ? 8 * ((k >> 2) & 1) : 0; }
    struct M32 {
        static constexpr int SIDE = 32, KSTEP = 8, MFMAS = 4;
        typedef f32x4 Frag;
        typedef f32x16 Acc;
        __device__ static __forceinline__ Frag read_k(const char *row, int swz, int step, int g)
        {
            return *reinterpret_cast<const f32x4 *>(row + (((2 * step + g) ^ swz) * 16));
        }
        template <int RB> __device__ static __forceinline__ Frag read_mn(const char *tile, int lane, int col0, int step)
        {
            const int h = lane / 32, byte = (col0 + lane % 32) * 4;
            const char *ad = tile + (step * KSTEP + 4 * h) * RB + (((byte / 16) ^ mn_swz(4 * h, RB / 16)) * 16) + byte % 16;
            Frag f;
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const float *>(ad + i * RB);
            return f;
        }
        __device__ static __forceinline__ Acc mfma(Frag a, Frag b, Acc c, int i)
        {
            return __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[i], c, 0, 0, 0);
        }
    };
};

// How the four wavefronts make a 32 x 32 tile.  bf16, fp8: a 16 x 16 block each, so that an element's sum stays one chain.
// fp32: the whole tile each, over a quarter of the k-steps, the four partial sums added at the end: an MFMA
// takes twice as long for a sixteenth of the products, and the shorter chains' error is no larger.
template <typename E, int T> struct Instr {
    typedef typename E::M32 M;
    static constexpr int KW = 1;
};
template <> struct Instr<Bf16, 32> {
    typedef Bf16::M16 M;
    static constexpr int KW = 1;
};
template <> struct Instr<Fp8, 32> {
    typedef Fp8::M16 M;
    static constexpr int KW = 1;
};
template <> struct Instr<F32, 32> {
    typedef F32::M32 M;
    static constexpr int KW = 4;
};

// x / d = (x mul) >> shift
struct Divisor {
    uint64_t mul;
    int shift;
};

struct Params {
    const char *A, *B;
    char *C;
    int64_t sA, sB, sC;            // batch strides in bytes
    int Mo, No, Kc;
    int tiles_m, tiles_n, group_m;
    float alpha;
    int out_f32, out_wide;         // out_wide: 16-byte runs of output columns are aligned and lie in one shard
    GemmMaps maps;
    unsigned step_a, step_b;       // bytes from one K-tile to the next inside a shard
    int items;                     // gemm_ring.h: tiles of all blocks, and what an item's number is divided by
    Divisor by_tiles, by_group, by_last;
};

// What a product runs on: the tile side, the bytes per load that its sizes and distances allow (the kernels exist for
// 16, 4 and one element's), the kernel's arguments.  CUBE3D_ENOTIMPL: left to gemm_generic.
struct Plan {
    int tile, piece;
    Params params;
};
int make_plan(const GemmArgs &g, Plan *plan);

// The ring kernel's tile (gemm_ring.h) and the estimated time of the launch in us; tile_m = 0: not for that kernel.
struct RingPlan {
    int tile_m, tile_n;
    float us;
};
RingPlan ring_plan(const GemmArgs &g, const Plan &plan);
// Whether it writes the result with streaming stores.
bool ring_streams(const GemmArgs &g, const Params &p, const RingPlan &r);

constexpr int ring_ktile_bytes(int tile_n) { return tile_n == 32 ? 256 : 128; }
// Offsets of an operand element stay below RING_SPAN; ROW_OUT marks a row or column beyond the operand, K_OUT an index beyond
// the contraction: any sum with one of them (or both) lies in [RING_SPAN, 2^32).
constexpr unsigned RING_SPAN = 1u << 30, ROW_OUT = 1u << 30, K_OUT = 1u << 31;

template <int GB> struct Piece;
template <> struct Piece<16> { typedef i32x4 Type; };
template <> struct Piece<4> { typedef int Type; };
template <> struct Piece<2> { typedef unsigned short Type; };
template <> struct Piece<1> { typedef unsigned char Type; };

// One operand's share of a lane: which pieces it loads, where they go in LDS, and the walk.
template <typename E, int T, int GB, bool KM> struct Operand {
    typedef typename Piece<GB>::Type P;
    static constexpr int SUB = 16 / GB;                 // pieces per 16-byte slot
    static constexpr int EPS = 16 / E::ELT, EPP = GB / E::ELT;
    static constexpr int TK = BKB / E::ELT;
    static constexpr int NP = T * BKB / 16 / 256;       // slots per lane
    static constexpr int RB = KM ? BKB : T * E::ELT;    // bytes of an LDS row
    static constexpr int SPR = RB / 16;
    static constexpr int PASS = 256 / SPR;              // rows between a lane's slots
    static constexpr int NST = KM ? NP : SUB, NWK = KM ? SUB : NP;
    static constexpr int BYTES = T * BKB;

    static constexpr int NV = NP * SUB;

    const char *base;
    unsigned st[NST];          // byte offset of the output index
    unsigned o[NV];            // byte offset of the pieces of the K-tile that starts at k
    int k, in_shard;           // wave-uniform: that K-tile's first contraction index, its position in its shard
    int kfirst;                // contraction index of walk 0 inside a K-tile
    int lds;                   // LDS byte of slot 0

    __device__ __forceinline__ void place(const AxisMap &km, int Kc)
    {
        in_shard = k - (int)(((uint64_t)(unsigned)k * km.M2) >> km.N2) * km.P2;
#pragma unroll
        for (int w = 0; w < NWK; ++w) {
            // (beyond Kc the offset is not used)
            const unsigned off = (unsigned)(axis_offset_fast(km, min(k + kfirst + w * (KM ? EPP : PASS), Kc - 1)) * E::ELT);
#pragma unroll
            for (int s = 0; s < NST; ++s) o[KM ? s * SUB + w : w * SUB + s] = st[s] + off;
        }
    }

    __device__ __forceinline__ void init(const char *b, const AxisMap &mn, const AxisMap &km, int m0, int extent, int Kc, int tid)
    {
        base = b;
        const int row = tid / SPR, slot = tid % SPR;
        // (a lane's rows are PASS apart: a multiple of what the permutations depend on)
        static_assert(PASS % (KM || T == 32 ? 16 : 8) == 0, "the permutation is the same for a lane's slots");
        lds = row * RB + ((slot ^ (KM ? (row / 2) % 8 : E::mn_swz(row, SPR))) * 16);
        kfirst = KM ? slot * EPS : row;
#pragma unroll
        for (int i = 0; i < NST; ++i) {
            const int x = KM ? min(m0 + row + i * PASS, extent - 1) : min(m0 + slot * EPS + i * EPP, extent - EPP);
            st[i] = (unsigned)(axis_offset_fast(mn, x) * E::ELT);
        }
        k = 0;
        place(km, Kc);
    }

    // Load the K-tile that starts at k, then move on to the next one.  Unless a shard ends inside these two
    // K-tiles every piece moves by the same distance; the branch is wave-uniform and has no load behind it,
    // so that the waits before the LDS writes stay exact counts.
    template <bool TAIL> __device__ __forceinline__ void load(P (&v)[NV], const AxisMap &km, unsigned step, int Kc)
    {
#pragma unroll
        for (int i = 0; i < NP; ++i)
#pragma unroll
            for (int u = 0; u < SUB; ++u) {
                unsigned at = o[i * SUB + u];
                if (TAIL) at = k + kfirst + (KM ? u * EPP : i * PASS) < Kc ? at : 0;
                v[i * SUB + u] = *reinterpret_cast<const P *>(base + at);
            }
        k += TK;
        if (in_shard + 2 * TK <= km.P2) {
            in_shard += TK;
#pragma unroll
            for (int i = 0; i < NV; ++i) o[i] += step;
        } else place(km, Kc);
    }

    template <bool TAIL> __device__ __forceinline__ void store(const P (&v)[NV], char *tile, int k0, int Kc) const
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            struct alignas(16) Slot { P p[SUB]; } s;
#pragma unroll
            for (int u = 0; u < SUB; ++u) {
                s.p[u] = v[i * SUB + u];
                if (TAIL && k0 + kfirst + (KM ? u * EPP : i * PASS) >= Kc) s.p[u] = P{};
            }
            *reinterpret_cast<i32x4 *>(tile + lds + i * PASS * RB) = __builtin_bit_cast(i32x4, s);
        }
    }
};

// K-tiles of loads in flight, in registers (T / 4 per lane and K-tile in pieces of 4 bytes and more, one per piece in
// narrower ones): as many as the accumulators leave room for in pieces of 16 bytes.  Narrower pieces keep one K-tile, with an
// offset register each; more was not tried for the 4-byte kernels, which use 60-70 registers at T = 32, 94-125 at T = 64.
constexpr int depth(int T, int GB) { return GB < 16 ? 1 : T == 128 ? 2 : 4; }

template <typename E, int T, int GB, bool AK, bool BK>
__global__ __launch_bounds__(256, T == 128 || GB == 1 ? 2 : 3) void gemm_edge_kernel(const Params p)
{
    typedef Operand<E, T, GB, AK> OA;
    typedef Operand<E, T, GB, BK> OB;
    typedef typename Instr<E, T>::M M;
    typedef typename M::Frag Frag;
    typedef typename M::Acc Acc;
    constexpr int SIDE = M::SIDE, VALS = SIDE * SIDE / 64;      // an accumulator block and a lane's values of it
    constexpr int KW = Instr<E, T>::KW, W = KW == 1 ? T / 2 : T, NB = W / SIDE;
    constexpr int TK = OA::TK, STEPS = TK / M::KSTEP, D = depth(T, GB);
    constexpr int STAGE = OA::BYTES + OB::BYTES;
    constexpr int STRIP = W * 4 + 16;                   // bytes of a staged output row (fp32, padded)
    constexpr int LDS = 2 * STAGE > 4 * SIDE * STRIP ? 2 * STAGE : 4 * SIDE * STRIP;   // the strips reuse the K-tile buffers
    static_assert(STEPS % KW == 0, "whole k-steps per wavefront");
    __shared__ __attribute__((aligned(1024))) char smem[LDS];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = KW == 1 ? (wave >> 1) * W : 0, wn = KW == 1 ? (wave & 1) * W : 0, g = lane / SIDE, in_side = lane % SIDE;

    // Workgroup ids go round robin over the 8 XCDs: hand every XCD one contiguous run of tiles, so that the
    // panels its workgroups share come through one L2.
    const int total = gridDim.x, id = blockIdx.x, xcd = id % 8, each = total / 8, more = total % 8;
    const int item = xcd * each + min(xcd, more) + id / 8;
    const int tiles = p.tiles_m * p.tiles_n, batch = item / tiles, tile = item - batch * tiles;
    const int per_group = p.group_m * p.tiles_n, gid = tile / per_group, first_m = gid * p.group_m;
    const int gsz = min(p.tiles_m - first_m, p.group_m), in_group = tile - gid * per_group;
    const int m0 = (first_m + in_group % gsz) * T, n0 = (in_group / gsz) * T;

    OA a;
    OB b;
    a.init(p.A + batch * p.sA, p.maps.a_mn, p.maps.a_k, m0, p.Mo, p.Kc, tid);
    b.init(p.B + batch * p.sB, p.maps.b_mn, p.maps.b_k, n0, p.No, p.Kc, tid);
    typename OA::P va[D][OA::NV];
    typename OB::P vb[D][OB::NV];

    Acc acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < VALS; ++v) acc[i][j][v] = 0.f;

    auto frag_a = [&](const char *ta, int i, int step) -> Frag {
        if constexpr (AK) {
            const int row = wm + SIDE * i + in_side;
            return M::read_k(ta + row * BKB, (row / 2) % 8, step, g);
        } else return M::template read_mn<OA::RB>(ta, lane, wm + SIDE * i, step);
    };
    auto frag_b = [&](const char *ta, int j, int step) -> Frag {
        const char *tb = ta + OA::BYTES;
        if constexpr (BK) {
            const int row = wn + SIDE * j + in_side;
            return M::read_k(tb + row * BKB, (row / 2) % 8, step, g);
        } else return M::template read_mn<OB::RB>(tb, lane, wn + SIDE * j, step);
    };
    // The MFMAs of one K-tile, with `moves` (the LDS writes and loads of later K-tiles) behind the fragment
    // reads of the first EARLY steps: a wavefront that is alone on its SIMD has its MFMAs wait for those
    // reads only, and not for the writes.
    constexpr int MY_STEPS = STEPS / KW, EARLY = T == 128 ? 1 : MY_STEPS < 4 ? MY_STEPS : 4;
    constexpr bool MOVES_LAST = T == 128;
    auto compute = [&](const char *ta, auto &&moves) {
        Frag fa[EARLY][NB], fb[EARLY][NB];
        auto step_no = [&](int s) { return KW == 1 ? s : wave * MY_STEPS + s; };
        auto read = [&](int s) {
#pragma unroll
            for (int i = 0; i < NB; ++i) fa[s % EARLY][i] = frag_a(ta, i, step_no(s));
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[s % EARLY][j] = frag_b(ta, j, step_no(s));
        };
#pragma unroll
        for (int s = 0; s < EARLY; ++s) read(s);
        if constexpr (!MOVES_LAST) moves();
#pragma unroll
        for (int s = 0; s < MY_STEPS; ++s) {
            if (s >= EARLY) read(s);
#pragma unroll
            for (int x = 0; x < M::MFMAS; ++x)      // (consecutive MFMAs on different accumulators where there are several)
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[i][j] = M::mfma(fb[s % EARLY][j], fa[s % EARLY][i], acc[i][j], x);
        }
        if constexpr (MOVES_LAST) moves();
    };

    const int full = p.Kc / TK, ntiles = (p.Kc + TK - 1) / TK;
    // K-tile kt travels in register set kt % D and sits in LDS buffer kt & 1.  The loop proper takes only
    // whole K-tiles and has no branch around a load, so that each wait covers one K-tile's loads and leaves the
    // younger ones in flight; the last K-tiles look at every piece's bounds (beyond the last one they load
    // element 0 and write zeros).
    auto load = [&](auto tail, int d) {
        a.template load<tail.value>(va[d], p.maps.a_k, p.step_a, p.Kc);
        b.template load<tail.value>(vb[d], p.maps.b_k, p.step_b, p.Kc);
    };
    // (an even number of K-tiles per pass: buffer and LDS addresses are constants)
    auto buffer = [&](int d, int kt) { return smem + (D % 2 == 0 ? d & 1 : kt & 1) * STAGE; };
    auto store = [&](auto tail, int d, int kt) {
        char *t = buffer(d, kt);
        a.template store<tail.value>(va[d], t, kt * TK, p.Kc);
        b.template store<tail.value>(vb[d], t + OA::BYTES, kt * TK, p.Kc);
    };
    const std::integral_constant<bool, false> whole{};
    const std::integral_constant<bool, true> tail{};
#pragma unroll
    for (int d = 0; d < D; ++d) load(tail, d);
    store(tail, 0, 0);
    load(tail, 0);
    __syncthreads();
    int k0 = 0;
    for (; k0 + 2 * D < full; k0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            // (the buffer of K-tile kt + 1 was last read before the previous barrier)
            const int kt = k0 + d;
            compute(buffer(d, kt), [&] {
                store(whole, (d + 1) % D, kt + 1);
                load(whole, (d + 1) % D);
            });
            __syncthreads();
        }
    }
    for (; k0 < ntiles; k0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int kt = k0 + d;
            if (kt < ntiles)
                compute(buffer(d, kt), [&] {
                    store(tail, (d + 1) % D, kt + 1);
                    load(tail, (d + 1) % D);
                });
            __syncthreads();
        }
    }

    // Output.  A lane's accumulator holds row lane % SIDE and columns 8 (v / 4) + 4 (lane / SIDE) + v % 4 of its
    // block (operands exchanged in the MFMA): one strip of SIDE rows at a time goes through LDS as fp32 so that
    // a lane stores 16 consecutive bytes of a row.  Where four wavefronts share the tile their strips are
    // added in ascending order, each wavefront a quarter of the rows.
    char *strip = smem + wave * SIDE * STRIP;
    const int run = p.out_f32 ? 4 : 8;                   // columns per 16-byte store
    const int lpr = W / run;                             // lanes per row: a power of two
    const int lcol = (lane % lpr) * run, col = n0 + wn + lcol;
    float bias[8];
    const bool has_bias = p.maps.bias != nullptr;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        bias[e] = (has_bias && e < run && col + e < p.No) ? p.maps.bias[axis_offset_fast(p.maps.bias_n, col + e)] : 0.f;
    const int es = p.out_f32 ? 4 : 2;
    char *C = p.C + batch * p.sC;
    const int64_t col_off = col < p.No ? axis_offset_fast(p.maps.c_n, col) : 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < VALS; v += 4) {
                f32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = acc[i][j][v + e];
                *reinterpret_cast<f32x4 *>(strip + in_side * STRIP + (SIDE * j + 2 * v + 4 * g) * 4) = w;
            }
        __syncthreads();
        const int r_first = KW == 1 ? 0 : wave * (SIDE / KW), r_end = r_first + SIDE / KW;
        for (int r = r_first + lane / lpr; r < r_end; r += 64 / lpr) {
            const int row = m0 + wm + SIDE * i + r;
            if (row >= p.Mo || col >= p.No) continue;
            const int64_t row_off = axis_offset_fast(p.maps.c_m, row);
            float x[8];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half && p.out_f32) break;
                const char *src = (KW == 1 ? strip : smem) + r * STRIP + lcol * 4 + half * 16;
                f32x4 t = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
                for (int k = 1; k < KW; ++k) t += *reinterpret_cast<const f32x4 *>(src + k * SIDE * STRIP);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * half + e] = t[e] * p.alpha + bias[4 * half + e];
            }
            if (p.out_wide) {
                char *dst = C + (row_off + col_off) * es;
                if (p.out_f32) *reinterpret_cast<f32x4 *>(dst) = f32x4{x[0], x[1], x[2], x[3]};
                else *reinterpret_cast<i32x4 *>(dst) = i32x4{(int)pack_bf16x2(x[0], x[1]), (int)pack_bf16x2(x[2], x[3]),
                                                             (int)pack_bf16x2(x[4], x[5]), (int)pack_bf16x2(x[6], x[7])};
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e < run && col + e < p.No) {
                        const int64_t at = row_off + axis_offset_fast(p.maps.c_n, col + e);
                        if (p.out_f32) reinterpret_cast<float *>(C)[at] = x[e];
                        else reinterpret_cast<unsigned short *>(C)[at] = f32_to_bf16_bits(x[e]);
                    }
            }
        }
        __syncthreads();
    }
}

// ---- host side --------------------------------------------------------------------------------------------

template <typename E, int T, int GB> int launch_layout(const GemmArgs &g, const Params &p)
{
    const dim3 grid((unsigned)((int64_t)p.tiles_m * p.tiles_n * g.batch)), block(256);
    if (g.a_kmajor && g.b_kmajor) hipLaunchKernelGGL((gemm_edge_kernel<E, T, GB, true, true>), grid, block, 0, g.stream, p);
    else if (g.a_kmajor) hipLaunchKernelGGL((gemm_edge_kernel<E, T, GB, true, false>), grid, block, 0, g.stream, p);
    else hipLaunchKernelGGL((gemm_edge_kernel<E, T, GB, false, false>), grid, block, 0, g.stream, p);
    return launch_status();
}

template <typename E, int GB> int launch_tile(const GemmArgs &g, const Params &p, int tile)
{
    if constexpr (GB > 1) {     // (single bytes: the pieces of a 128 x 128 tile don't fit the registers)
        if (tile == 128) return launch_layout<E, 128, GB>(g, p);
    }
    return tile == 32 ? launch_layout<E, 32, GB>(g, p) : launch_layout<E, 64, GB>(g, p);
}

}  // namespace edge

// per element type, in a translation unit of its own (piece = bytes per load as chosen by gemm_edge)
int gemm_edge_bf16(const GemmArgs &g, const edge::Params &p, int tile, int piece);
int gemm_edge_fp8(const GemmArgs &g, const edge::Params &p, int tile, int piece);
int gemm_edge_f32(const GemmArgs &g, const edge::Params &p, int tile, int piece);
int gemm_ring_bf16(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r);
int gemm_ring_fp8(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r);
int gemm_ring_fp8_deep(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r);
int gemm_ring_f32(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r);

}  // namespace cube3d
