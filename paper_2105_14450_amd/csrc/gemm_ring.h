// Products of any size whose operands can be read in 16-byte pieces, for gfx950: the tiles of gemm_edge.h fetched straight
// into LDS.  bf16, fp8-e4m3 and fp32, plain leading dimensions or a cube of shards read in place.
//
// Work split.  A workgroup of eight wavefronts makes TM x TN tiles, one after the other: four wavefronts load (direct to
// LDS, into a ring of NST stages of one K-tile each), four multiply, one of either on every SIMD.  A direct-to-LDS load holds
// its wavefront up until the CU's 64 bytes per cycle have room for it, 64 cycles with four wavefronts loading: wavefronts
// that also multiply leave the matrix cores idle meanwhile, and the load path while they multiply.  2032 x 512 x 2048
// bf16, both operands K-major, tiles of 64: 12.4 us without loaders, 9.0-9.8 with, 13.8-15.0 in gemm_edge.h.  The loaders run
// on into the next tile while the output of the last one is stored, as far as the ring's stages go: vmcnt counts stores too, so
// the multipliers' first barrier behind an output waits until it has left.
//
// What bounds it (bf16, cycles per 128 bytes of contraction at 2.3 GHz).  Tiles of 64: the load path, 256 of 300.  Tiles of
// 128: 512 for the loads and 512 for the MFMAs, 700.  256 x 128: MFMAs, 1024 of 1150-1250, and one or a few tiles per CU.
// 8000 x 8192 x 2048: 225-240 us = 1.12-1.19 PFLOP/s, 318-329 in gemm_edge.h; three fp8 products of 3000 x 3072 x 12288
// 356-361 us = 1.9 PFLOP/s against 597.  Few rows (64 x 8192 x 2048 14.7 -> 11, 64 x 2048 x 8192 23 -> 22): one workgroup's K loop.
// fp8 operands with 256-byte LDS rows (MN-major, tiles 256 wide) are read with two-way bank conflicts: Fp8::mn_swz deals
// consecutive k-rows out for rows of 128 bytes.
//
// Edges.  The loads go through a buffer descriptor of 1 GiB: an offset beyond it reads as zeros, so rows beyond the
// output, indices beyond the contraction and K-tiles beyond the last one are loads like any other, and the number of loads
// in flight, which the waits count, never depends on the sizes.
//
// Addresses.  A lane's offset is a constant (its row or column, its place inside a K-tile); the offset of the K-tile's first
// contraction index is the load's scalar offset, looked up for 64 K-tiles at a time, one per lane.  Where a shard of the
// contraction index ends inside a K-tile, the lanes behind the end take the next shard's offset instead: one compare
// and one select per load, no branch.  At most one end may lie inside a K-tile (the dispatch checks it).
//
// Sums.  As in gemm_edge.h: all products of an element in ascending order in one accumulator (fp32: four of every eight
// indices alternately), and the same bits.  fp8 with bf16 results takes the 64-deep MFMA in tiles of 128 and more, twice as
// fast, with its operands laid out so that it adds in that order too (Fp8Deep).
#pragma once
#include "gemm_edge.h"

namespace cube3d {
namespace edge {

// fp8 with the 64-deep MFMA.  It adds 16 products at a time: the lower 16 bytes of lanes 0-31, those of lanes 32-63, then
// the upper 16 bytes of either.  Dealt out in that order the contraction indices are added as by four 16-deep MFMAs, to the
// last bit (524288 sums of 64, 512 and 4096 products of random bytes: none differs; with a run of 32 indices per lane half
// 2, 19 and 62 % of them do), so a row's bits do not depend on the tile here either.
struct Fp8Deep {
    static constexpr int ELT = 1;
    __device__ static __forceinline__ int mn_swz(int k, int spr) { return Fp8::mn_swz(k, spr); }
    struct M32 {
        static constexpr int SIDE = 32, KSTEP = 64, MFMAS = 1;
        typedef i32x8 Frag;
        typedef f32x16 Acc;
        __device__ static __forceinline__ Frag read_k(const char *row, int swz, int step, int g)
        {
            const int c = 4 * step + g;
            const i32x4 lo = *reinterpret_cast<const i32x4 *>(row + ((c ^ swz) * 16));
            const i32x4 hi = *reinterpret_cast<const i32x4 *>(row + (((c + 2) ^ swz) * 16));
            return Frag{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
        template <int RB> __device__ static __forceinline__ Frag read_mn(const char *tile, int lane, int col0, int step)
        {
            const int g = lane / 16;
            Frag f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const i32x2 v = Fp8::read_mn_at<RB>(tile + step * KSTEP * RB, lane % 16, col0 + 16 * (g % 2), 32 * (i / 2) + 16 * (g / 2) + 8 * (i % 2));
                f[2 * i] = v[0];
                f[2 * i + 1] = v[1];
            }
            return f;
        }
        __device__ static __forceinline__ Acc mfma(Frag a, Frag b, Acc c, int)
        {
            return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
        }
    };
};

// Direct-to-LDS 16-byte load: lane s of the wavefront writes LDS bytes [lds + 16 s, +16) with the 16 bytes at `offset` of
// the buffer, zeros if that lies beyond it.  Inline assembly, so that its completion is tracked by the ring's own waits
// and by nothing else (the compiler would drain every load before each LDS read).
__device__ __forceinline__ void ring_load(i32x4 buffer, unsigned offset, unsigned scalar_offset, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %3 offen lds" : : "v"(offset), "s"(buffer), "s"(lds), "s"(scalar_offset) : "m0");
}

// At most N of this wavefront's loads and no LDS read outstanding.
template <int N> __device__ __forceinline__ void ring_wait()
{
    // gfx9 encoding: vmcnt = bits 3:0 and 15:14, expcnt = bits 6:4, lgkmcnt = bits 11:8
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

// At most N of this wavefront's loads and none of its LDS reads outstanding, then meet the others.  The empty asm
// statements keep LDS accesses on their side of the barrier.
template <int N> __device__ __forceinline__ void ring_barrier()
{
    asm volatile("" ::: "memory");
    ring_wait<N>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The last NST barriers of a loader, or all if there are fewer: the K-tiles in flight become fewer.
template <int NST, int LPT, int D = 0> __device__ __forceinline__ void ring_drain(int barriers)
{
    if constexpr (D < NST) {
        if (D < barriers) ring_barrier<(D + 2 < NST ? NST - 2 - D : 0) * LPT>();
        ring_drain<NST, LPT, D + 1>(barriers);
    }
}

// A value that a vector instruction left in a scalar register, through the scalar unit: 5 wait states lie between the former
// and a vector memory instruction that reads it only where the compiler sees one, which it does not in ring_load.  (The build
// refuses an assembly where any load is nearer, to a spilled register for instance.  5 wait states in ring_load itself
// took 118.8 us for three fp32 products of 2048 x 512 x 2048 in place of 115.9.)
__device__ __forceinline__ unsigned scalar(unsigned x)
{
    unsigned y;
    asm volatile("s_mov_b32 %0, %1" : "=s"(y) : "s"(x));
    return y;
}

// Place of index x inside its shard (a prepared map).
__device__ __forceinline__ int place_in_shard(const AxisMap &m, int x) { return x - (int)(((uint64_t)(unsigned)x * m.M2) >> m.N2) * m.P2; }

// One operand's share of a wavefront: where its lanes read, and the walk along the contraction index.
template <typename E, int T, int BKB, bool KM> struct RingOperand {
    static constexpr int EPS = 16 / E::ELT, TK = BKB / E::ELT;
    static constexpr int RB = KM ? BKB : T * E::ELT, SPR = RB / 16;      // an LDS row, its 16-byte slots
    static constexpr int RPC = 1024 / RB, ROWS = 4 * RPC;                 // rows per load of a wavefront, of the workgroup
    static constexpr int BYTES = T * BKB, LOADS = BYTES / 4096;           // per wavefront and K-tile
    static_assert(RPC >= 1 && LOADS >= 1 && BYTES % 4096 == 0, "whole 1 KB pieces of LDS per wavefront");

    __device__ static __forceinline__ int swz(int row)
    {
        // 16 consecutive rows of a K-major tile at one slot lie in 16 different slots modulo 256 bytes
        return KM ? (BKB == 256 ? row % 16 : (row / 2) % 8) : E::mn_swz(row, SPR);
    }

    i32x4 buffer;
    unsigned lane_off[LOADS];
    int kin;                       // contraction index inside a K-tile: of all loads (K-major), of the first one
    // of K-tile `lane` of the current 64: offset of its first contraction index, indices before the end of the shard or of
    // the contraction, what the lanes behind that end take instead
    unsigned at, behind;
    int limit;

    __device__ __forceinline__ void init(const char *base, const AxisMap &mn, const AxisMap &km, int m0, int extent, int wave, int lane)
    {
        const uint64_t b = (uint64_t)base;
        buffer = i32x4{(int)b, (int)(b >> 32) & 0xffff, (int)RING_SPAN, 0x00020000};
        const int row = wave * RPC + lane / SPR, slot = (lane % SPR) ^ swz(row);
        static_assert(KM ? ROWS % 16 == 0 : ROWS % 16 == 0 || (ROWS % 8 == 0 && SPR >= (E::ELT == 1 ? 8 : 16)), "the permutation is the same for all loads of a lane");
        kin = KM ? slot * EPS : row;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int x = KM ? m0 + row + i * ROWS : m0 + slot * EPS;
            const unsigned off = (unsigned)(axis_offset_fast(mn, min(x, extent - 1)) * E::ELT);
            lane_off[i] = (x < extent ? off : ROW_OUT) + (unsigned)(kin + (KM ? 0 : i * ROWS)) * (unsigned)(km.u * E::ELT);
        }
    }

    // K-tiles first ... first + 63; whether K-tile `lane` of them lies in one shard
    __device__ __forceinline__ bool look_ahead(const AxisMap &km, int Kc, int first, int lane)
    {
        const int k0 = (first + lane) * TK, rem = Kc - k0;
        const int shard = (int)(((uint64_t)(unsigned)min(k0, Kc - 1) * km.M2) >> km.N2), left = (shard + 1) * km.P2 - k0;
        limit = min(rem, left);
        at = rem > 0 ? (unsigned)(axis_offset_fast(km, k0) * E::ELT) : K_OUT;
        behind = rem > left ? (unsigned)((axis_offset_fast(km, k0 + left) - left * km.u) * E::ELT) : K_OUT;
        return limit >= TK;
    }

    // Load K-tile `t` of the current 64 into the stage at LDS byte `lds` (this wavefront's share of it): one that lies in
    // one shard, or any
    __device__ __forceinline__ void load_one_shard(int t, unsigned lds) const
    {
        const unsigned k = scalar((unsigned)__builtin_amdgcn_readlane((int)at, t));
#pragma unroll
        for (int i = 0; i < LOADS; ++i) ring_load(buffer, lane_off[i], k, lds + i * 4096);
    }

    __device__ __forceinline__ void load_any(int t, unsigned lds) const
    {
        const unsigned k = __builtin_amdgcn_readlane((int)at, t), next = __builtin_amdgcn_readlane((int)behind, t);
        const int end = __builtin_amdgcn_readlane(limit, t);
#pragma unroll
        for (int i = 0; i < LOADS; ++i) ring_load(buffer, lane_off[i] + (kin + (KM ? 0 : i * ROWS) < end ? k : next), 0, lds + i * 4096);
    }
};

// Which tile an item is.
struct Place {
    int batch, m0, n0;
};

__device__ __forceinline__ int divide(int x, const Divisor &d) { return (int)(((uint64_t)(unsigned)x * d.mul) >> d.shift); }

__device__ __forceinline__ Place place_item(const Params &p, int id, int TM, int TN)
{
    // Items go round robin over the 8 XCDs (a workgroup's next item is a multiple of 8 away): hand every XCD one contiguous
    // run of tiles, so that the panels its workgroups share come through one L2.
    const int xcd = id % 8, each = p.items / 8, more = p.items % 8, item = xcd * each + min(xcd, more) + id / 8;
    const int tiles = p.tiles_m * p.tiles_n, batch = p.items == tiles ? 0 : divide(item, p.by_tiles), tile = item - batch * tiles;
    const int gid = divide(tile, p.by_group), first_m = gid * p.group_m, in_group = tile - gid * p.group_m * p.tiles_n;
    const int gsz = min(p.tiles_m - first_m, p.group_m);
    const int col = gsz == p.group_m ? in_group / 8 : divide(in_group, p.by_last);
    return Place{batch, (first_m + in_group - col * gsz) * TM, col * TN};
}

// The matrix instruction of a tile, the bytes of a K-tile per row, the stages of the ring.
template <typename E, int T> struct RingInstr { typedef typename E::M32 M; };
template <> struct RingInstr<Bf16, 32> { typedef Bf16::M16 M; };
template <> struct RingInstr<Fp8, 32> { typedef Fp8::M16 M; };

// Output of a wavefront's blocks, JH of them side by side at a time through a strip of LDS of its own: a lane's accumulator
// holds row lane % SIDE and columns 8 (v / 4) + 4 (lane / SIDE) + v % 4 of a block (operands exchanged in the MFMA) and
// stores 16 consecutive bytes of a row.  The 16-byte slots of a strip row are permuted by the row, so that neither side has
// bank conflicts.
template <typename M, int NBM, int NBN, int OES, bool BIAS, bool STREAM> struct RingOutput {
    static constexpr int SIDE = M::SIDE, VALS = SIDE * SIDE / 64;
    static constexpr int JH = OES == 2 && NBN % 2 == 0 ? 2 : 1;
    static constexpr int ROWB = JH * SIDE * OES, LPR = ROWB / 16, RPP = 64 / LPR < SIDE ? 64 / LPR : SIDE;    // bytes and lanes of a strip row, rows per pass
    static constexpr int BYTES = SIDE * ROWB;
    static constexpr bool LARGEST = NBM * NBN > 4;      // tiles above 128 x 128

    __device__ static __forceinline__ int perm(int row) { return (row * ROWB / 256) % LPR; }

    __device__ static __forceinline__ void store(const Params &p, const typename M::Acc (&acc)[NBM][NBN], char *strip, int m0, int n0, int batch, int lane)
    {
        // (opaque: formed ahead of the K loop, the addresses below would occupy registers all through it)
        asm volatile("" : "+v"(lane));
        const int g = lane / SIDE, in_side = lane % SIDE, rd_row = lane / LPR, rd_slot = lane % LPR;
        char *C = p.C + batch * p.sC;
        const int64_t row_step = p.maps.c_m.u;
#pragma unroll
        for (int jh = 0; jh < NBN; jh += JH) {
            const int col = n0 + jh * SIDE + rd_slot * (16 / OES);
            const int64_t col_off = col < p.No ? axis_offset_fast(p.maps.c_n, col) : 0;
            // the bias of this lane's columns, by way of the strip
            f32x4 bias[JH][VALS / 4];
            if constexpr (BIAS) {
                if (lane < JH * SIDE) {
                    const int c = n0 + jh * SIDE + lane;
                    reinterpret_cast<float *>(strip)[lane] = c < p.No ? p.maps.bias[axis_offset_fast(p.maps.bias_n, c)] : 0.f;
                }
#pragma unroll
                for (int j = 0; j < JH; ++j)
#pragma unroll
                    for (int v = 0; v < VALS; v += 4)
                        bias[j][v / 4] = *reinterpret_cast<const f32x4 *>(strip + (j * SIDE + 2 * v + 4 * g) * 4);
            }
#pragma unroll
            for (int i = 0; i < NBM; ++i) {
#pragma unroll
                for (int j = 0; j < JH; ++j)
#pragma unroll
                    for (int v = 0; v < VALS; v += 4) {
                        float x[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = acc[i][jh + j][v + e] * p.alpha + (BIAS ? bias[j][v / 4][e] : 0.f);
                        const int byte = (j * SIDE + 2 * v + 4 * g) * OES;
                        char *dst = strip + in_side * ROWB + (((byte / 16) ^ perm(in_side)) * 16) + byte % 16;
                        if constexpr (OES == 4) *reinterpret_cast<f32x4 *>(dst) = f32x4{x[0], x[1], x[2], x[3]};
                        else *reinterpret_cast<i32x2 *>(dst) = i32x2{(int)pack_bf16x2(x[0], x[1]), (int)pack_bf16x2(x[2], x[3])};
                    }
                // largest tiles: the strip's rows mostly lie in one shard, then one division does for all of them
                const int first = m0 + i * SIDE;
                const bool one_shard = LARGEST && place_in_shard(p.maps.c_m, first) + SIDE <= p.maps.c_m.P2;
                const int64_t first_off = one_shard ? axis_offset_fast(p.maps.c_m, first) : 0;
                if (p.out_wide) {
#pragma unroll
                    for (int ps = 0; ps < SIDE / RPP; ++ps) {
                        const int r = ps * RPP + rd_row, row = first + r;
                        const i32x4 x = *reinterpret_cast<const i32x4 *>(strip + r * ROWB + ((rd_slot ^ perm(r)) * 16));
                        if (row >= p.Mo || col >= p.No || r >= SIDE) continue;
                        const int64_t row_off = one_shard ? first_off + r * row_step : axis_offset_fast(p.maps.c_m, row);
                        i32x4 *dst = reinterpret_cast<i32x4 *>(C + (row_off + col_off) * OES);
                        if (STREAM) __builtin_nontemporal_store(x, dst);
                        else *dst = x;
                    }
                } else {        // element by element, rolled up: the instruction cache holds 64 KB
#pragma unroll 1
                    for (int r = rd_row; r < SIDE; r += RPP) {
                        if (first + r >= p.Mo) break;
                        const int64_t row_off = axis_offset_fast(p.maps.c_m, first + r);
                        const char *src = strip + r * ROWB + ((rd_slot ^ perm(r)) * 16);
#pragma unroll 1
                        for (int e = 0; e < 16 / OES && col + e < p.No; ++e) {
                            char *dst = C + (row_off + axis_offset_fast(p.maps.c_n, col + e)) * OES;
                            if constexpr (OES == 4) *reinterpret_cast<int *>(dst) = *reinterpret_cast<const int *>(src + 4 * e);
                            else *reinterpret_cast<unsigned short *>(dst) = *reinterpret_cast<const unsigned short *>(src + 2 * e);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);      // (one strip at a time: else registers for all of them)
            }
        }
    }
};

// bytes of LDS: the ring, and a strip per wavefront that holds a block of the output in fp32 or two in bf16
constexpr int ring_strip(int TN) { return TN == 32 ? 16 * 16 * 4 : 32 * 32 * 4; }
constexpr int ring_lds(int TM, int TN, int NST) { return NST * (TM + TN) * ring_ktile_bytes(TN) + 4 * ring_strip(TN); }
constexpr int ring_per_cu(int TM, int TN, int NST) { return ring_lds(TM, TN, NST) > 80 * 1024 ? 1 : 2; }

// Persistent workgroups: workgroup w makes the tiles w, w + gridDim.x, ...  STREAM: streaming stores of the output.
template <typename E, int TM, int TN, int NST, bool AK, bool BK, bool STREAM>
__global__ __launch_bounds__(512, 2 * ring_per_cu(TM, TN, NST)) void gemm_ring_kernel(const Params p)
{
    constexpr int BKB = ring_ktile_bytes(TN);
    typedef RingOperand<E, TM, BKB, AK> OA;
    typedef RingOperand<E, TN, BKB, BK> OB;
    typedef typename RingInstr<E, TM>::M M;
    typedef typename M::Frag Frag;
    typedef typename M::Acc Acc;
    constexpr int SIDE = M::SIDE, VALS = SIDE * SIDE / 64, WM = TM / 2, WN = TN / 2, NBM = WM / SIDE, NBN = WN / SIDE;
    constexpr int STEPS = OA::TK / M::KSTEP;
    // Fragments are read one unit ahead: a K-tile, or a k-step of the largest tiles, whose accumulators leave less room.
    constexpr int USTEPS = TM * TN > 128 * 128 ? 1 : STEPS, UNITS = STEPS / USTEPS;
    constexpr int STAGE = OA::BYTES + OB::BYTES, LPT = OA::LOADS + OB::LOADS;
    static_assert(UNITS == 1 || UNITS % 2 == 0, "the fragment buffers alternate per unit");
    static_assert((NST - 1) * LPT <= 63, "vmcnt range");
    constexpr int STRIP = ring_strip(TN);
    static_assert(RingOutput<M, NBM, NBN, 2, false, STREAM>::BYTES <= STRIP && RingOutput<M, NBM, NBN, 4, false, STREAM>::BYTES <= STRIP, "room for the output strips");
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, 4> I4;
    __shared__ __attribute__((aligned(1024))) char smem[ring_lds(TM, TN, NST)];

    const int tid = threadIdx.x, lane = tid & 63, wave8 = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wave8 % 4;
    const int ntiles = (p.Kc + OA::TK - 1) / OA::TK, my_items = (p.items - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;

    // K-tile c (counted over all items of the workgroup) sits in stage c % NST.  Behind barrier c, K-tile c + 1 has landed and
    // everybody has the fragments of c: K-tile c + NST goes to their stage.
    if (wave8 >= 4) {
        OA a;
        OB b;
        const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)smem + wave * 1024;
        uint64_t one_shard = 0;        // bit t: K-tile t of the current 64 lies in one shard of either operand
        int item = blockIdx.x, kt = 0;                  // next K-tile to load
        unsigned to = lds0;                             // and its stage
        auto start_item = [&]() {
            const Place at = place_item(p, item, TM, TN);
            a.init(p.A + at.batch * p.sA, p.maps.a_mn, p.maps.a_k, at.m0, p.Mo, wave, lane);
            b.init(p.B + at.batch * p.sB, p.maps.b_mn, p.maps.b_k, at.n0, p.No, wave, lane);
        };
        auto next_stage = [&]() { to = to + STAGE == lds0 + NST * STAGE ? lds0 : to + STAGE; };
        // any K-tile (behind the last item: beyond the contraction, zeros)
        auto load = [&]() {
            const int t = kt % 64;
            if (t == 0) {
                const bool whole_a = a.look_ahead(p.maps.a_k, p.Kc, kt, lane), whole_b = b.look_ahead(p.maps.b_k, p.Kc, kt, lane);
                one_shard = __ballot(whole_a && whole_b);
            }
            a.load_any(t, to);
            b.load_any(t, to + OA::BYTES);
            next_stage();
            if (++kt == ntiles && item + (int)gridDim.x < p.items) {
                item += gridDim.x;
                kt = 0;
                start_item();
            }
        };
        start_item();
#pragma unroll 1
        for (int s = 0; s < NST - 1; ++s) load();
        ring_barrier<(NST - 2) * LPT>();      // K-tile 0 is there
        load();
        const int total = ntiles * my_items;
        int left = total - NST;        // K-tiles still to load
        while (left > 0) {
            // a run of K-tiles in one shard each, but not the first of 64 or the last of the item
            const int t = kt % 64;
            int run = t == 0 ? 0 : min(min(__builtin_ctzll(~(one_shard >> t) | 1ull << (64 - t)), ntiles - 1 - kt), left);
            left -= run;
            kt += run;
            for (int u = t; run > 0; --run, ++u) {
                ring_barrier<(NST - 2) * LPT>();
                a.load_one_shard(u, to);
                b.load_one_shard(u, to + OA::BYTES);
                next_stage();
            }
            if (left > 0) {
                ring_barrier<(NST - 2) * LPT>();
                load();
                --left;
            }
        }
        ring_drain<NST, LPT>(total);
        ring_wait<0>();     // (fewer K-tiles than stages) nothing may arrive behind the workgroup's end
        return;
    }

    const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN, g = lane / SIDE, in_side = lane % SIDE;
    char *strip = smem + NST * STAGE + wave * STRIP;
    Acc acc[NBM][NBN];
    Frag fa[2][USTEPS][NBM], fb[2][USTEPS][NBN];
    int stage = 0;
    // fragment r of a unit, A and B alternately in the order in which the MFMAs need them
    constexpr int FRAGS = USTEPS * (NBM + NBN);
    auto read = [&](int r, int buf, const char *ta, int unit) {
        const char *tb = ta + OA::BYTES;
        const int s = r / (NBM + NBN), x = r % (NBM + NBN), step = unit * USTEPS + s;
        if (x == 0 || x > NBN) {
            const int i = x == 0 ? 0 : x - NBN;
            if constexpr (AK) fa[buf][s][i] = M::read_k(ta + (wm + in_side) * BKB + i * SIDE * BKB, OA::swz(in_side), step, g);
            else fa[buf][s][i] = M::template read_mn<OA::RB>(ta, lane, wm + SIDE * i, step);
        } else {
            const int j = x - 1;
            if constexpr (BK) fb[buf][s][j] = M::read_k(tb + (wn + in_side) * BKB + j * SIDE * BKB, OB::swz(in_side), step, g);
            else fb[buf][s][j] = M::template read_mn<OB::RB>(tb, lane, wn + SIDE * j, step);
        }
    };
    // The MFMAs of a unit, with the reads of the next one ahead of them (one accumulator: the MFMAs wait for each other
    // anyway) or dealt out behind them, all but the last few.
    constexpr int MFMAS = USTEPS * M::MFMAS * NBM * NBN, GAPS = NBM * NBN == 1 ? 0 : MFMAS > 8 ? MFMAS - 4 : MFMAS > 4 ? MFMAS - 2 : MFMAS;
    auto multiply = [&](int buf, const char *next, int next_unit) {
        if constexpr (GAPS == 0) {
#pragma unroll
            for (int r = 0; r < FRAGS; ++r) read(r, buf ^ 1, next, next_unit);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MFMAS; ++m) {
            const int s = m / (M::MFMAS * NBM * NBN), x = m / (NBM * NBN) % M::MFMAS, i = m / NBN % NBM, j = m % NBN;
            acc[i][j] = M::mfma(fb[buf][s][j], fa[buf][s][i], acc[i][j], x);
            if constexpr (GAPS > 0) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < FRAGS; ++r)
                    if (r * GAPS / FRAGS == m) read(r, buf ^ 1, next, next_unit);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    const std::true_type yes{};
    const std::false_type no{};
    // K-tile with its first unit's fragments in buffer `buf`; moves to the next stage
    auto k_tile = [&](auto buf_c) {
        constexpr int buf = decltype(buf_c)::value;
        const char *here = smem + stage * STAGE;
#pragma unroll
        for (int u = 0; u < UNITS - 1; ++u) multiply((buf + u) & 1, here, u + 1);
        __builtin_amdgcn_sched_barrier(0);
        ring_barrier<0>();
        stage = stage + 1 == NST ? 0 : stage + 1;
        multiply((buf + UNITS - 1) & 1, smem + stage * STAGE, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    ring_barrier<0>();
    for (int item = blockIdx.x; item < p.items; item += gridDim.x) {
#pragma unroll
        for (int i = 0; i < NBM; ++i)
#pragma unroll
            for (int j = 0; j < NBN; ++j)
#pragma unroll
                for (int v = 0; v < VALS; ++v) acc[i][j][v] = 0.f;
#pragma unroll
        for (int r = 0; r < FRAGS; ++r) read(r, 0, smem + stage * STAGE, 0);
        if constexpr (UNITS == 1) {
            for (int kt = 0; kt < ntiles; kt += 2) {
                k_tile(std::integral_constant<int, 0>{});
                if (kt + 1 < ntiles) k_tile(std::integral_constant<int, 1>{});
            }
        } else {
            for (int kt = 0; kt < ntiles; ++kt) k_tile(std::integral_constant<int, 0>{});
        }
        const Place at = place_item(p, item, TM, TN);
        auto store = [&](auto oes, auto bias) {
            RingOutput<M, NBM, NBN, decltype(oes)::value, decltype(bias)::value, STREAM>::store(p, acc, strip, at.m0 + wm, at.n0 + wn, at.batch, lane);
        };
        // (a bias comes with the layout of the forward product, K-major times MN-major)
        if (AK && !BK && p.maps.bias != nullptr) p.out_f32 ? store(I4{}, yes) : store(I2{}, yes);
        else p.out_f32 ? store(I4{}, no) : store(I2{}, no);
    }
}

// ---- host side --------------------------------------------------------------------------------------------

// (as the multipliers of an index map: exact for numbers below 2^31)
inline Divisor make_divisor(int d)
{
    AxisMap m{d, d, 0, 0, 1};
    prepare_axis_map(m);
    return Divisor{m.M1, m.N1};
}

template <typename E, int TM, int TN, int NST> int ring_layout(const GemmArgs &g, Params p)
{
    p.tiles_m = (p.Mo + TM - 1) / TM;
    p.tiles_n = (p.No + TN - 1) / TN;
    const int64_t items = (int64_t)p.tiles_m * p.tiles_n * g.batch;
    const int64_t places = (int64_t)num_compute_units() * ring_per_cu(TM, TN, NST) / 8 * 8;
    if (items >= (1ll << 31) - places || places < 8) return CUBE3D_ENOTIMPL;
    p.items = (int)items;
    p.group_m = 8;
    p.by_tiles = make_divisor(p.tiles_m * p.tiles_n);
    p.by_group = make_divisor(p.group_m * p.tiles_n);
    p.by_last = make_divisor(p.tiles_m % p.group_m ? p.tiles_m % p.group_m : p.group_m);
    const dim3 grid((unsigned)(items < places ? items : places)), block(512);
    auto launch = [&](auto stream) {
        constexpr bool S = decltype(stream)::value;
        if (g.a_kmajor && g.b_kmajor) hipLaunchKernelGGL((gemm_ring_kernel<E, TM, TN, NST, true, true, S>), grid, block, 0, g.stream, p);
        else if (g.a_kmajor) hipLaunchKernelGGL((gemm_ring_kernel<E, TM, TN, NST, true, false, S>), grid, block, 0, g.stream, p);
        else hipLaunchKernelGGL((gemm_ring_kernel<E, TM, TN, NST, false, false, S>), grid, block, 0, g.stream, p);
        return launch_status();
    };
    if constexpr (TM * TN > 128 * 128) {
        if (ring_streams(g, p, RingPlan{TM, TN, 0.f})) return launch(std::true_type{});
    }
    return launch(std::false_type{});
}

template <typename E> int ring_small(const GemmArgs &g, const Params &p, const RingPlan &r)
{
    if constexpr (E::ELT < 4) {
        if (r.tile_m == 32) return ring_layout<E, 32, 32, 4>(g, p);
    }
    return ring_layout<E, 64, 64, 4>(g, p);
}

template <typename E> int ring_large(const GemmArgs &g, const Params &p, const RingPlan &r)
{
    if constexpr (E::ELT < 4) {
        if (r.tile_m == 256) return ring_layout<E, 256, 128, 3>(g, p);
        if (r.tile_n == 256) return ring_layout<E, 128, 256, 3>(g, p);
    }
    return ring_layout<E, 128, 128, 4>(g, p);
}

template <typename E> int ring_any(const GemmArgs &g, const Params &p, const RingPlan &r)
{
    return r.tile_m < 128 ? ring_small<E>(g, p, r) : ring_large<E>(g, p, r);
}

}  // namespace edge
}  // namespace cube3d
