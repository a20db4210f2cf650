// Instantiations of the ring kernel (gemm_ring.h): fp8 operands, with the 16- and 32-deep MFMAs.
#include "gemm_ring.h"

namespace cube3d {

int gemm_ring_fp8(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r)
{
    return edge::ring_any<edge::Fp8>(g, p, r);
}

}  // namespace cube3d
