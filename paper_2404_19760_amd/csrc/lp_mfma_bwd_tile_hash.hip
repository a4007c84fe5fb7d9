// The tile kernels of the Renderer's backward (lp_mfma_bwd_tile.h) over hash tables: windows are taken on
// the virtual lattice, each of whose texels adds into its table entry.  Table of 2^19 x 16 over a 128^3 lattice, 128^2
// rays x 128 samples (8 adds of a line per sample one ray at a time): 0.69 ms with one wave per ray (lp_mfma_bwd.h)
// -> 0.457 ms.
#include "lp_mfma_bwd_tile.h"

namespace lp {

hipError_t launch_bwd_tile_hash(const GridDev& g, const MlpDev& m, const RaysDev& rays, const BwdIo& io, int n_cu,
                           hipStream_t stream)
{
    return dispatch_bwd_tile<LP_GRID_HASH>(g, m, rays, io, n_cu, stream);
}

}  // namespace lp
