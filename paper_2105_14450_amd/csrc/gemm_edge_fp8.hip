// Instantiations of the product kernel for any size (gemm_edge.h): fp8 operands.
#include "gemm_edge.h"

namespace cube3d {

int gemm_edge_fp8(const GemmArgs &g, const edge::Params &p, int tile, int piece)
{
    if (piece >= 16) return edge::launch_tile<edge::Fp8, 16>(g, p, tile);
    if (piece >= 4) return edge::launch_tile<edge::Fp8, 4>(g, p, tile);
    return edge::launch_tile<edge::Fp8, 1>(g, p, tile);
}

}  // namespace cube3d
