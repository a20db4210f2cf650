// Instantiations of the product kernel for any size (gemm_edge.h): fp32 operands.
#include "gemm_edge.h"

namespace cube3d {

int gemm_edge_f32(const GemmArgs &g, const edge::Params &p, int tile, int piece)
{
    if (piece >= 16) return edge::launch_tile<edge::F32, 16>(g, p, tile);
    return edge::launch_tile<edge::F32, 4>(g, p, tile);
}

}  // namespace cube3d
