// Instantiations of the ring kernel (gemm_ring.h): fp32 operands.
#include "gemm_ring.h"

namespace cube3d {

int gemm_ring_f32(const GemmArgs &g, const edge::Params &p, const edge::RingPlan &r)
{
    return edge::ring_any<edge::F32>(g, p, r);
}

}  // namespace cube3d
