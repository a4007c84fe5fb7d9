// Matrix-core backward kernel of the Renderer: dispatch and most instantiations (see
// lp_mfma_bwd.h).
#include "lp_mfma_bwd.h"

#include <cstdlib>

namespace lp {

namespace {

// 16 grid channels + direction inputs (the two-MLP decoder merged into one MLP of 32 inputs); with contract
// coordinates, and the widest variant on a triplane: the other translation unit
template <int KIND>
hipError_t dispatch_bwd(const GridDev& g, const MlpDev& m, const RaysDev& rays, const BwdIo& io, int n_cu,
                         hipStream_t stream)
{
    const int C = m.dims[0], CG = g.C, H = m.dims[1], NH = m.n_layers - 1;
    if (C != 32 || CG != 16) return hipErrorInvalidValue;
    if (g.contract > 0.0 || (KIND == LP_GRID_TRIPLANE && H == 64 && NH == 2))
        return launch_bwd_mfma_b(g, m, rays, io, n_cu, stream);
#define LP_CASE(h, nh) \
    if (H == h && NH == nh) return launch_bwd<KIND, 32, h, nh, false, 16, kAnyDtype>(g, m, rays, io, n_cu, stream);
    LP_CASE(32, 1) LP_CASE(64, 1) LP_CASE(32, 2)
    if constexpr (KIND == LP_GRID_VOXEL) { LP_CASE(64, 2) }
#undef LP_CASE
    return hipErrorInvalidValue;
}

}  // namespace

// one workgroup of 4 waves per compute unit, rounded up to a multiple of the 8 XCDs
int mfma_bwd_records(int n_cu) { return ((n_cu + 7) / 8 * 8) * kWaves; }

hipError_t launch_bwd_mfma(const GridDev& g, const MlpDev& m, const RaysDev& rays, const BwdIo& io, int n_cu,
                           hipStream_t stream)
{
    // The tile kernels take every shape whose inputs are all grid channels. The older layouts of the largest
    // configuration's shape stay selectable when the library is loaded: LP_BWD_ONE_WAVE=1 (one wave per ray),
    // LP_BWD_TWO_WAVE=1 (a chain wave and a weights wave per ray).
    static const auto chosen = [](const char* name) { const char* e = std::getenv(name); return e && e[0] == '1'; };
    static const bool one_wave = chosen("LP_BWD_ONE_WAVE"), two_wave = chosen("LP_BWD_TWO_WAVE");
    if ((one_wave || two_wave) && bwd_ws_supported(g, m)) {
        if (two_wave) return launch_bwd_mfma_ws(g, m, rays, io, n_cu, stream);
        if (g.dtype == LP_BF16) return launch_bwd<LP_GRID_VOXEL, 16, 64, 2, false, 16, LP_BF16>(g, m, rays, io, n_cu, stream);
        if (g.dtype == LP_F16) return launch_bwd<LP_GRID_VOXEL, 16, 64, 2, false, 16, LP_F16>(g, m, rays, io, n_cu, stream);
        return g.contract > 0.0 ? launch_bwd<LP_GRID_VOXEL, 16, 64, 2, true, 16>(g, m, rays, io, n_cu, stream)
                                : launch_bwd<LP_GRID_VOXEL, 16, 64, 2, false, 16>(g, m, rays, io, n_cu, stream);
    }
    if (m.dims[0] == g.C) {
        if (g.kind == LP_GRID_VOXEL) return launch_bwd_tile_voxel(g, m, rays, io, n_cu, stream);
        if (g.kind == LP_GRID_TRIPLANE) return launch_bwd_tile_triplane(g, m, rays, io, n_cu, stream);
        if (g.kind == LP_GRID_HASH) return launch_bwd_tile_hash(g, m, rays, io, n_cu, stream);
    }
    if (g.kind == LP_GRID_HASH) return launch_bwd_mfma_hash(g, m, rays, io, n_cu, stream);
    if (g.kind == LP_GRID_HEXPLANE) return launch_bwd_mfma_hexplane(g, m, rays, io, n_cu, stream);
    return g.kind == LP_GRID_VOXEL ? dispatch_bwd<LP_GRID_VOXEL>(g, m, rays, io, n_cu, stream)
                                   : dispatch_bwd<LP_GRID_TRIPLANE>(g, m, rays, io, n_cu, stream);
}

}  // namespace lp
