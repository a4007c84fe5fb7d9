// Naive Splatter forward (Section 3.3 "Splatter": every point of a pixel's ray pushes the pixel's
// feature vector into the cell that contains it).
//
// What bounds it: the rate of atomic adds (2.1e10 64-byte lines/s on this chip). Pushed ray by ray, a point adds
// about 10 lines after runs in a cell are merged; a step is therefore a tile of four neighbouring rays, eight points
// of each, whose window of texels is summed as a matrix product of interpolation weights and pixel features
// (lp_tile_scatter.h) and added once per texel: 3.93 lines per point. The weight sums go to the one-channel structure
// by the lanes that hold the texels' weights. Rays that do not run side by side are pushed one after the other, 32
// points per step, by the run-merging walk.
// 160^3 x 32 voxels, 4 x 128^2 rays x 160 points: 5.41 ms ray by ray -> 2.18 ms (4.12e7 lines: 90 % of the rate of the adds).
// Tiles are visited in scrambled order like the Renderer's backward
// (atomic adds of neighbouring rays queue up at the same L2 channel).
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_mfma_bwd_common.h"
#include "lp_splat_common.h"
#include "lp_tile_scatter.h"

namespace lp {

namespace {

constexpr int kWaves = 4;
constexpr int kArea = kWinBytes;   // LDS of a wave: the window's table, or the records of a walk
static_assert(kArea >= 32 * 16 * 4, "the walk's records");

template <int KIND, int C, bool CC>
__global__ __launch_bounds__(kWaves * 64) void splat_naive_kernel(GridDev tgt, RaysDev rays, SplatDev sp, PushOrder order)
{
    __shared__ __align__(16) char areas[kWaves][kArea];
    const int lane = threadIdx.x & 63;
    const int col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)areas[wave];

    const int rays_per_item = order.tiles ? kTileRays : 1;
    const RaySchedule sched = ray_schedule(order.n_groups * kWaves, kWaves);
    const int S = rays.S;
    for (long long seq = sched.first; seq < sched.end; seq += sched.stride) {
        const long long first = (((seq / kWaves) * order.group_mul % order.n_groups) * kWaves + seq % kWaves) * rays_per_item;
        if (first >= rays.M) continue;
        const bool tile = order.tiles && side_by_side(rays, first, col, [&](const RayGeom& r, int j) { return sample_cell<CC>(tgt, r, j); });
        const int n_sub = tile ? 1 : (int)min((long long)rays_per_item, rays.M - first);
        for (int sub = 0; sub < n_sub; ++sub) {
            const long long r = first + (tile ? col / kTileSamples : sub);
            const bool ray_ok = r < rays.M;
            const RayGeom q = load_ray_geom(rays, min(r, rays.M - 1));
            const int scene = __builtin_amdgcn_readfirstlane(q.scene);
            // the pixels' features of this lane's channel (16 channels: both halves of a lane group)
            f32x16 val;
#pragma unroll
            for (int i = 0; i < kTileRays; ++i) {
                const long long at = min(first + (tile ? i : sub), rays.M - 1);
                const float v = sp.feats[(size_t)at * C + (col & (C - 1))];
#pragma unroll
                for (int e = 0; e < 4; ++e) val[4 * i + e] = v;
            }
            const int step = tile ? kTileSamples : 32, k = tile ? col % kTileSamples : col;
            for (int j0 = 0; j0 < S; j0 += step) {
                const int j = j0 + k;
                const Cell3 c = sample_cell<CC>(tgt, q, min(j, S - 1));
                scatter_step<KIND, C, Scatter::kPushRay>(tgt, sp.theta, scene, area, areas[wave], c, val, lane, tile,
                                                         sp.theta_w, ray_ok && j < S);
            }
        }
    }
}

template <int KIND, int C, bool CC>
hipError_t launch(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    long long blocks = 4LL * n_cu;   // four workgroups per compute unit
    blocks = (blocks + 7) / 8 * 8;
    const PushOrder order = push_order(rays, blocks * kWaves, kWaves);
    if (blocks > order.n_groups) blocks = (order.n_groups + 7) / 8 * 8;
    hipLaunchKernelGGL((splat_naive_kernel<KIND, C, CC>), dim3((unsigned)blocks), dim3(kWaves * 64), 0, stream, tgt,
                       rays, sp, order);
    return hipGetLastError();
}

template <int KIND>
hipError_t dispatch(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    const bool cc = tgt.contract > 0.0;
    if (tgt.C == 16) return cc ? launch<KIND, 16, true>(tgt, rays, sp, n_cu, stream) : launch<KIND, 16, false>(tgt, rays, sp, n_cu, stream);
    if (tgt.C == 32) return cc ? launch<KIND, 32, true>(tgt, rays, sp, n_cu, stream) : launch<KIND, 32, false>(tgt, rays, sp, n_cu, stream);
    return hipErrorInvalidValue;
}

}  // namespace

bool splat_naive_supported(const GridDev& tgt)
{
    if (tgt.kind != LP_GRID_VOXEL && tgt.kind != LP_GRID_TRIPLANE && tgt.kind != LP_GRID_HASH) return false;
    if (tgt.C != 16 && tgt.C != 32) return false;
    if (tgt.kind == LP_GRID_HASH) {   // a table whose size is a power of two (`mod size` is a mask in this kernel)
        const unsigned long long T = tgt.hash_size;
        return T != 0 && (T & (T - 1)) == 0 && T * tgt.C < (1ull << 30);
    }
    const unsigned long long n0 = (unsigned long long)tgt.N[0], n1 = (unsigned long long)tgt.N[1], n2 = (unsigned long long)tgt.N[2];
    if (tgt.kind == LP_GRID_VOXEL) return n0 * n1 * n2 * tgt.C < (1ull << 30);   // 32-bit byte offsets in a scene
    return n0 * n1 * tgt.C < (1ull << 30) && n1 * n2 * tgt.C < (1ull << 30) && n2 * n0 * tgt.C < (1ull << 30);
}

hipError_t launch_splat_naive(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu,
                              hipStream_t stream)
{
    if (tgt.kind == LP_GRID_HASH) return dispatch<LP_GRID_HASH>(tgt, rays, sp, n_cu, stream);
    return tgt.kind == LP_GRID_VOXEL ? dispatch<LP_GRID_VOXEL>(tgt, rays, sp, n_cu, stream)
                                     : dispatch<LP_GRID_TRIPLANE>(tgt, rays, sp, n_cu, stream);
}

}  // namespace lp
