// Prints which kernel family, tile side and load width the library picks for products, one per line of standard input:
//   plain <dtype> <out dtype> <a K-major> <b K-major> <batch> <Mo> <No> <Kc>
//   cube  <dtype> <out dtype> <op: 0 forward, 1 dX, 2 dW> <q> <M> <K> <N>           (input gathered along y, no bias)
// One line of output each, host code only: nothing is launched.
//   tile piece      of the any-size kernel through registers, "0 0" where it leaves the product to the element-wise one
//   rows columns    tile of the ring kernel, "0 0" where that does not take the product in its place
//   wide stream     whether output runs of 16 bytes are stored whole, and whether the ring kernel streams them
//   tuned           tile side of the tile-aligned kernel, which comes before all of these, or 0
#include <stdio.h>
#include <string.h>

#include "gemm_edge.h"

using namespace cube3d;

static AxisMap cut(int64_t p1, int64_t p2, int64_t s1, int64_t s2, int64_t u)
{
    return AxisMap{(int32_t)p1, (int32_t)p2, s1, s2, u};
}

int main()
{
    char kind[16];
    int dtype, out;
    while (scanf("%15s %d %d", kind, &dtype, &out) == 3) {
        GemmArgs g{};
        GemmMaps m{};
        g.in_dtype = dtype;
        g.out_dtype = out;
        g.alpha = 1.f;
        if (!strcmp(kind, "plain")) {
            int ak, bk;
            long long mo, no, kc;
            if (scanf("%d %d %d %lld %lld %lld", &ak, &bk, &g.batch, &mo, &no, &kc) != 6) return 1;
            g.a_kmajor = ak; g.b_kmajor = bk;
            g.Mo = mo; g.No = no; g.Kc = kc;
            g.lda = ak ? kc : mo; g.ldb = bk ? kc : no; g.ldc = no;
            g.strideA = mo * kc; g.strideB = no * kc; g.strideC = mo * no;
        } else {
            int op;
            long long q, M, K, N;
            if (scanf("%d %lld %lld %lld %lld", &op, &q, &M, &K, &N) != 5) return 1;
            // X shards [M/q^2, K/q], W shards [K/q, N/q^2], Y shards [M/q^2, N/q]; processor (i, a, b) has number (i q + a) q + b
            const long long Mb = M / q, Kb = K / q, Nb = N / q, Ms = Mb / q, Ns = Nb / q, q2 = q * q;
            const long long x = Ms * Kb, w = Kb * Ns, y = Ms * Nb;
            const AxisMap xm = cut(Mb, Ms, q2 * x, q * x, Kb), xk = cut(Kb, Kb, x, 0, 1);
            const AxisMap wk = cut(Kb, Kb, w, 0, Ns), wn = cut(Nb, Ns, q * w, q2 * w, 1);
            const AxisMap ym = cut(Mb, Ms, q2 * y, y, Nb), yn = cut(Nb, Nb, q * y, 0, 1);
            g.batch = 1;
            g.a_kmajor = op != 2;
            g.b_kmajor = op == 1;
            if (op == 0) { g.Mo = M; g.No = N; g.Kc = K; m.a_mn = xm; m.a_k = xk; m.b_mn = wn; m.b_k = wk; m.c_m = ym; m.c_n = yn; }
            if (op == 1) { g.Mo = M; g.No = K; g.Kc = N; m.a_mn = ym; m.a_k = yn; m.b_mn = wk; m.b_k = wn; m.c_m = xm; m.c_n = xk; }
            if (op == 2) { g.Mo = K; g.No = N; g.Kc = M; m.a_mn = xk; m.a_k = xm; m.b_mn = yn; m.b_k = ym; m.c_m = wk; m.c_n = wn; }
            m.bias_n = m.c_n;
            g.maps = &m;
        }
        edge::Plan plan;
        const bool taken = edge::make_plan(g, &plan) == CUBE3D_OK;
        edge::RingPlan ring{0, 0, 0.f};
        if (taken) ring = edge::ring_plan(g, plan);
        printf("%d %d %d %d %d %d %d\n", taken ? plan.tile : 0, taken ? plan.piece : 0, ring.tile_m, ring.tile_n,
               taken && plan.params.out_wide, ring.tile_m > 0 && edge::ring_streams(g, plan.params, ring), gemm_fast_plan(g).tile);
    }
    return 0;
}
