// Instantiations of the ring kernel (gemm_ring.h): fp8 operands, with the 64-deep MFMAs.
#include "gemm_ring.h"

namespace cube3d {

int gemm_ring_fp8_deep(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r)
{
    return edge::ring_large<edge::Fp8Deep>(g, p, r);
}

}  // namespace cube3d
