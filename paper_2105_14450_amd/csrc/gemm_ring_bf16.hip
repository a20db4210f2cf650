// Instantiations of the ring kernel (gemm_ring.h): bf16 operands.
#include "gemm_ring.h"

namespace cube3d {

int gemm_ring_bf16(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r)
{
    return edge::ring_any<edge::Bf16>(g, p, r);
}

}  // namespace cube3d
