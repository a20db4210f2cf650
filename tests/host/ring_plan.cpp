// Prints the tile of the ring kernel for products on plain operands, one per line of standard input:
//   <dtype> <out dtype> <a K-major> <b K-major> <batch> <Mo> <No> <Kc>
// One line of output each: "rows columns", or "0 0" where another kernel takes the product.  Host code only.
#include <stdio.h>

#include "gemm_edge.h"

using namespace cube3d;

int main()
{
    int ak, bk;
    long long mo, no, kc;
    GemmArgs g{};
    while (scanf("%d %d %d %d %d %lld %lld %lld", &g.in_dtype, &g.out_dtype, &ak, &bk, &g.batch, &mo, &no, &kc) == 8) {
        g.alpha = 1.f;
        g.a_kmajor = ak; g.b_kmajor = bk;
        g.Mo = mo; g.No = no; g.Kc = kc;
        g.lda = ak ? kc : mo; g.ldb = bk ? kc : no; g.ldc = no;
        g.strideA = mo * kc; g.strideB = no * kc; g.strideC = mo * no;
        edge::Plan plan;
        edge::RingPlan ring{0, 0, 0.f};
        if (edge::make_plan(g, &plan) == CUBE3D_OK) ring = edge::ring_plan(g, plan);
        printf("%d %d\n", ring.tile_m, ring.tile_n);
    }
    return 0;
}
