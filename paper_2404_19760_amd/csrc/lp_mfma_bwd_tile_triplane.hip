// The tile kernels of the Renderer's backward (lp_mfma_bwd_tile.h) over triplanes.
#include "lp_mfma_bwd_tile.h"

namespace lp {

hipError_t launch_bwd_tile_triplane(const GridDev& g, const MlpDev& m, const RaysDev& rays, const BwdIo& io, int n_cu,
                           hipStream_t stream)
{
    return dispatch_bwd_tile<LP_GRID_TRIPLANE>(g, m, rays, io, n_cu, stream);
}

}  // namespace lp
