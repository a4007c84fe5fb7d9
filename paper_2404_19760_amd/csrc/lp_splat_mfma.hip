// Splatter forward with an MLP on the matrix cores (Section 3.3 "Splatter": each point of a
// pixel's ray pushes g_s(pixel feature, prior structure sampled at the point, encoded
// direction) into the target structure).
//
// A step is 32 points: a tile of four neighbouring rays, eight points of each, or 32 points of one ray.  The MLP runs
// transposed like the Renderer's (hidden layers D = W X with the points along N).  The pixel feature and the direction encoding
// are the same for every point of a ray, so their part of the first layer, W1[:, per-ray inputs] x, is evaluated once per
// item, for the four rays side by side, and is the accumulator that a step's first layer starts from; it then contracts the
// prior's channels (gathered per point) only.  The last layer is taken
// with the roles swapped, V = H^T Wout^T (points along M, channels along N), which leaves lane =
// channel and registers = points: the layout that the scatter of a tile works on (lp_tile_scatter.h).  Contract coordinates are a
// run-time branch in the point placement (uniform over the launch).
// What bounds it: the atomic adds.  160^3 x 32 voxels, prior alike, MLP 67-64-64-32, 4 x 64^2 rays x 160 points: ray by ray
// 9.6 lines per point, 1.41 ms at 86 % of the rate of the adds; in tiles 5.25 lines, 0.76 ms at 86 %.
// Tiles where the launch is large enough (push_order) and the rays run in tiles; both kernels are launched and find out which is meant,
// 5 us.  Without the look rays that do not run side by side went one after the other through the tiles' kernel: push of 48^2 pixels
// three and four texels apart 0.69 .. 1.05 of the speed before tiles (0.89 .. 1.06 now), of 2304 rays in random order 0.78 .. 1.14 (0.90 ..
// 1.47).  Time of a forward before tiles over that now, 32^2 .. 176^2 pixels, 24 to 160 points, both structures, 16 and 32 channels:
// up to one texel from pixel to pixel 1.0 .. 3.9, at two 0.87 .. 2.0 (the slowest at 48^2 x 24 points, 103 -> 118 us), at three and
// four 0.88 .. 1.12, rays in random order 0.97 .. 1.46.
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_mfma_bwd_common.h"
#include "lp_splat_common.h"
#include "lp_tile_scatter.h"

#include <algorithm>

namespace lp {

namespace {

constexpr int kWaves = 4;
constexpr int kHidden = 64;

// LDS layout in 16-byte units.  KSP K-steps of prior channels (16 each), KSE K-steps of per-ray
// inputs (pixel feature, direction encoding, zeros); element e of lane group g in K-step s is
// input 16 s + 8 g + e of its kind.
template <int KSP, int KSE, int NH>
struct SplatLds {
    static constexpr int MB = kHidden / 32, KSH = kHidden / 16;
    static constexpr int A1P = 0;                                   // W1, prior columns   [MB][KSP]
    static constexpr int A1E = A1P + MB * KSP * 128;                // W1, per-ray columns [MB][KSE]
    static constexpr int A2 = A1E + MB * KSE * 128;                 // W2   [MB][KSH]  (NH == 2)
    static constexpr int A3 = A2 + (NH == 2 ? MB * KSH * 128 : 0);  // Wout as B operand [1][KSH]
    static constexpr int BIAS = A3 + KSH * 128;                     // floats b1[64] b2[64] bout[32]
    static constexpr int WAVE = BIAS + (2 * kHidden + 32) / 4;      // per-wave areas
    // a wave's area: the scatter's, and its four rays' 48 inputs
    static constexpr int W_X = kWinBytes / 16, W_UNITS = W_X + kTileRays * 48 / 4;
    static constexpr int UNITS = WAVE + kWaves * W_UNITS;
    static_assert(2 * (UNITS * 16 + 16) <= 160 * 1024, "two workgroups fit the LDS of a compute unit");
};

template <int KSP, int KSE, int NH, int CO>
__device__ __forceinline__ void stage_splat_mlp(uint4* lds, const MlpDev& m, int n_in)
{
    using L = SplatLds<KSP, KSE, NH>;
    constexpr int MB = L::MB, KSH = L::KSH, CP = 16 * KSP;
    auto hidden_col = [](int s, int gg, int e) { return k_hidden(s, gg, e); };
    auto block_row = [](int mb, int i) { return 32 * mb + i; };
    const int n_extra = n_in + m.n_enc;
    // the caller's column order is pixel feature, prior channels, direction encoding
    stage_operand(lds + L::A1P, m.W[0], MB, KSP, m.dims[0], block_row,
                  [=](int s, int gg, int e) { return n_in + 16 * s + 8 * gg + e; });
    stage_operand(lds + L::A1E, m.W[0], MB, KSE, m.dims[0], block_row, [=](int s, int gg, int e) {
        const int x = 16 * s + 8 * gg + e;
        return x < n_in ? x : x < n_extra ? CP + x : -1;
    });
    if constexpr (NH == 2) stage_operand(lds + L::A2, m.W[1], MB, KSH, kHidden, block_row, hidden_col);
    // last layer as the B operand of the swapped product: "row" i = output channel (16 channels:
    // a second copy in rows 16..31, both halves of a lane group scatter)
    stage_operand(lds + L::A3, m.W[NH], 1, KSH, kHidden, [](int, int i) { return i & (CO - 1); }, hidden_col);
    float* sbias = reinterpret_cast<float*>(lds + L::BIAS);
    for (int i = threadIdx.x; i < kHidden; i += blockDim.x) {
        sbias[i] = m.b[0][i];
        sbias[kHidden + i] = NH == 2 ? m.b[1][i] : 0.0f;
    }
    if (threadIdx.x < 32) sbias[2 * kHidden + threadIdx.x] = m.b[NH][threadIdx.x & (CO - 1)];
}

// Scatter of 32 points of one ray, column c = point slot_to_sample(c): a window where the whole step fits one (`windows`: it may), else
// the walk of run-merged records.
template <int KIND, int C>
__device__ __forceinline__ void push_ray_step(const GridDev& g, const SplatDev& sp, int scene, uint32_t area, char* area_ptr, const Cell3& cell,
                                              f32x16& v, int lane, bool valid, bool windows)
{
    const int col = lane & 31, grp = lane >> 5;
    if (windows) {
        float probe = 0.0f;   // (a product would spread an infinite vector over its window)
#pragma unroll
        for (int r = 0; r < 16; ++r) probe = fmaf(v[r], 0.0f, probe);
        const Window win = find_window(cell, true);
        if (window_fits<KIND>(win) && __ballot(probe != 0.0f) == 0ull) {
            scatter_window<KIND, C, Scatter::kPushPoints>(g, sp.theta, sp.theta_w, scene, area, win, cell, valid, v, lane);
            return;
        }
    }
    float* info = reinterpret_cast<float*>(area_ptr);
    wave_lds_fence();
    if (grp == 0) {
        float* rec = info + col * 16;
        write_scatter_record<KIND, C, true>(rec, g, cell);
        if (!valid) {   // a point past the end of the ray pushes nothing
#pragma unroll
            for (int k = 0; k < (KIND == LP_GRID_VOXEL ? 8 : 12); ++k) rec[k] = 0.0f;
        }
    }
    const unsigned there = (unsigned)__ballot(valid);
    if (there != 0xffffffffu) {   // (weight zero alone would turn an infinite vector into an undefined one)
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = ((there >> d_row(r, grp)) & 1u) ? v[r] : 0.0f;
    }
    wave_lds_fence();
    scatter_channels<KIND, C>(g, sp.theta, scene, info, v, col, grp);
    scatter_weights<KIND, C>(g, sp.theta_w, scene, info, col, grp);
}

// TILES: items are tiles of four rays (those that do not lie side by side go one after the other), else single rays.  `choose`: both
// kernels are launched, and the one that the rays suit works.
template <int KIND, int KSP, int KSE, int NH, bool TILES>
__global__ __launch_bounds__(kWaves * 64, 2) void splat_mfma_kernel(GridDev tgt, MlpDev m, RaysDev rays, SplatDev sp, PushOrder order, bool choose)
{
    if (choose && rays_run_in_tiles(tgt, rays, (float)kPushApart, 1e30f) != TILES) return;
    constexpr int CO = 16 * KSP;  // the target has the prior's channel count
    using L = SplatLds<KSP, KSE, NH>;
    constexpr int MB = L::MB, KSH = L::KSH;
    extern __shared__ uint4 lds[];
    stage_splat_mlp<KSP, KSE, NH, CO>(lds, m, sp.n_in);
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int col = lane & 31, grp = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint4* wave_area = lds + L::WAVE + wave * L::W_UNITS;
    char* const area_ptr = reinterpret_cast<char*>(wave_area);
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)area_ptr;
    float* ray_x = reinterpret_cast<float*>(wave_area + L::W_X);   // [4][48]
    const float* sbias = reinterpret_cast<const float*>(lds + L::BIAS);
    const float bias_out = sbias[2 * kHidden + col];
    const int n_in = sp.n_in, n_extra = sp.n_in + m.n_enc;

    constexpr int rays_per_item = TILES ? kTileRays : 1;
    const RaySchedule sched = ray_schedule(order.n_groups * kWaves, kWaves);
    const int S = rays.S;
    for (long long seq = sched.first; seq < sched.end; seq += sched.stride) {
        const long long first = (((seq / kWaves) * order.group_mul % order.n_groups) * kWaves + seq % kWaves) * rays_per_item;
        if (first >= rays.M) continue;
        const long long end = min(first + rays_per_item, rays.M);
        const bool tile = TILES && side_by_side<kPushApart>(rays, min(first + col / kTileSamples, end - 1), [&](const RayGeom& r, int j) { return sample_cell_any(tgt, r, j); });
        const int n_sub = tile ? 1 : (int)(end - first);
        for (int sub = 0; sub < n_sub; ++sub) {
            const long long ray = first + (tile ? col / kTileSamples : sub);
            const bool ray_ok = ray < end;
            const RayGeom q = load_ray_geom(rays, min(ray, end - 1));
            const int scene = __builtin_amdgcn_readfirstlane(q.scene);
            // ---- the rays' inputs x (pixel feature, direction encoding, zeros), one per lane, and the first layer's
            //      accumulators b1 + W1[:, per-ray inputs] x of the rays' columns ----
            f32x16 start[MB][1];
            {
                wave_lds_fence();
#pragma unroll
                for (int i = 0; i < kTileRays; ++i) {
                    if (i > 0 && !tile) break;
                    const long long at = min(first + (tile ? i : sub), end - 1);
                    const float d[3] = {rays.dirs[3 * at], rays.dirs[3 * at + 1], rays.dirs[3 * at + 2]};
                    const float x_lane = lane < n_in ? sp.feats[(size_t)at * n_in + lane]
                                                     : lane < n_extra ? dir_encoding(d, lane - n_in) : 0.0f;
                    if (lane < 48) ray_x[48 * i + lane] = x_lane;
                }
                wave_lds_fence();
                init_bias<MB, 1>(start, sbias, grp);
                const float* mine = ray_x + (tile ? 48 * (col / kTileSamples) : 0);
                Frag eh[1][KSE], el[1][KSE];
#pragma unroll
                for (int s = 0; s < KSE; ++s) {
                    float x[8];
                    *reinterpret_cast<f32x4*>(x) = *reinterpret_cast<const f32x4*>(mine + 16 * s + 8 * grp);
                    *reinterpret_cast<f32x4*>(x + 4) = *reinterpret_cast<const f32x4*>(mine + 16 * s + 8 * grp + 4);
                    split8(x, eh[0][s], el[0][s]);
                }
                layer_mfma<MB, KSE, 1>(start, lds + L::A1E, lane, eh, el);
            }
            const int step = tile ? kTileSamples : 32, k = tile ? col % kTileSamples : TILES ? col : slot_to_sample(col);
            bool windows = true;   // single rays: whether a step may fit a window
            if constexpr (!TILES) {
                const Cell3 c0 = sample_cell_any(tgt, q, 0), c1 = sample_cell_any(tgt, q, S - 1);
#pragma unroll
                for (int a = 0; a < 3; ++a) windows = windows && (long long)abs(c1.i[a] - c0.i[a]) * min(32, S) <= (long long)kWinExtent * S;
            }
            for (int j0 = 0; j0 < S; j0 += step) {
                const int j = j0 + k, jj = min(j, S - 1);
                Frag fh[1][KSP], fl[1][KSP];
                {
                    const Cell3 cp = sample_cell_any(sp.prior, q, jj);
#pragma unroll
                    for (int s = 0; s < KSP; ++s) {
                        float feat[8];
                        gather_half<KIND, CO, 8, LP_F32>(sp.prior, scene, cp, 16 * s + 8 * grp, feat);
                        split8(feat, fh[0][s], fl[0][s]);
                        __builtin_amdgcn_sched_barrier(0);   // one K-step's loads at a time
                    }
                }
                Frag lh[1][KSH], ll[1][KSH];
                {
                    f32x16 acc[MB][1];
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[mb][0] = start[mb][0];
                    layer_mfma<MB, KSP, 1>(acc, lds + L::A1P, lane, fh, fl);
                    to_operands<MB, true, 1>(acc, lh, ll);
                    if constexpr (NH == 2) {
                        init_bias<MB, 1>(acc, sbias + kHidden, grp);
                        layer_mfma<MB, KSH, 1>(acc, lds + L::A2, lane, lh, ll);
                        to_operands<MB, true, 1>(acc, lh, ll);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                // V[point][channel]: the hidden activations are the A operand as they stand
                f32x16 v;
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = bias_out;
#pragma unroll
                for (int s = 0; s < KSH; ++s) {
                    Frag wh, wl;
                    load_operand(lds + L::A3 + s * 128, lane, wh, wl);
                    v = mfma3(lh[0][s], ll[0][s], wh, wl, v);
                }
                __builtin_amdgcn_sched_barrier(0);
                uint32_t lane_here = lane;   // (or what the scatter derives from the lane number is kept through the loop)
                refresh(lane_here);
                const Cell3 cell = sample_cell_any(tgt, q, jj);
                const bool valid = ray_ok && j < S;
                if constexpr (TILES) scatter_step<KIND, CO, Scatter::kPushPoints, RayWindows::kWhole>(tgt, sp.theta, scene, area, area_ptr, cell, v, lane_here, step, sp.theta_w, valid);
                else push_ray_step<KIND, CO>(tgt, sp, scene, area, area_ptr, cell, v, lane_here, valid, windows);
            }
        }
    }
}

long long waves_of(int n_cu) { return (2LL * n_cu + 7) / 8 * 8 * kWaves; }

template <int KIND, int KSP, int KSE, int NH>
hipError_t launch(const GridDev& tgt, const MlpDev& m, const RaysDev& rays, const SplatDev& sp, int n_cu,
                  hipStream_t stream)
{
    constexpr int kLdsBytes = SplatLds<KSP, KSE, NH>::UNITS * 16;
    const PushOrder tiles = push_order(rays, waves_of(n_cu), kWaves), single = push_order(rays, waves_of(n_cu), kWaves, 0.0);
    auto start = [&](auto kernel, const PushOrder& order) {
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
        const long long blocks = std::min(waves_of(n_cu) / kWaves, (order.n_groups + 7) / 8 * 8);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kWaves * 64), kLdsBytes, stream, tgt, m, rays, sp, order, tiles.tiles != 0);
        return hipGetLastError();
    };
    if (tiles.tiles) {
        const hipError_t e = start(splat_mfma_kernel<KIND, KSP, KSE, NH, true>, tiles);
        if (e != hipSuccess) return e;
    }
    return start(splat_mfma_kernel<KIND, KSP, KSE, NH, false>, single);
}

template <int KIND, int KSP, int KSE>
hipError_t by_layers(const GridDev& tgt, const MlpDev& m, const RaysDev& rays, const SplatDev& sp, int n_cu,
                     hipStream_t stream)
{
    return m.n_layers == 2 ? launch<KIND, KSP, KSE, 1>(tgt, m, rays, sp, n_cu, stream)
                           : launch<KIND, KSP, KSE, 2>(tgt, m, rays, sp, n_cu, stream);
}

template <int KIND, int KSP>
hipError_t by_extras(const GridDev& tgt, const MlpDev& m, const RaysDev& rays, const SplatDev& sp, int n_cu,
                     hipStream_t stream)
{
    const int n_extra = sp.n_in + m.n_enc;
    if (n_extra <= 16) return by_layers<KIND, KSP, 1>(tgt, m, rays, sp, n_cu, stream);
    if (n_extra <= 32) return by_layers<KIND, KSP, 2>(tgt, m, rays, sp, n_cu, stream);
    return by_layers<KIND, KSP, 3>(tgt, m, rays, sp, n_cu, stream);
}

template <int KIND>
hipError_t by_channels(const GridDev& tgt, const MlpDev& m, const RaysDev& rays, const SplatDev& sp, int n_cu,
                       hipStream_t stream)
{
    return tgt.C == 16 ? by_extras<KIND, 1>(tgt, m, rays, sp, n_cu, stream)
                       : by_extras<KIND, 2>(tgt, m, rays, sp, n_cu, stream);
}

}  // namespace

bool splat_mfma_supported(const GridDev& tgt, const MlpDev& m, const SplatDev& sp)
{
    if (tgt.kind != LP_GRID_VOXEL && tgt.kind != LP_GRID_TRIPLANE) return false;   // (hash tables: generic kernels)
    if (m.n_layers != 2 && m.n_layers != 3) return false;
    for (int l = 1; l < m.n_layers; ++l)
        if (m.dims[l] != kHidden) return false;
    if (!sp.has_prior || sp.prior.C != tgt.C || sp.prior.dtype != LP_F32) return false;
    if (tgt.contract != sp.prior.contract) return false;
    if (sp.n_in + m.n_enc > 48) return false;
    return splat_naive_supported(tgt) && splat_naive_supported(sp.prior);
}

hipError_t launch_splat_mfma(const GridDev& tgt, const MlpDev& m, const RaysDev& rays, const SplatDev& sp,
                             int n_cu, hipStream_t stream)
{
    return tgt.kind == LP_GRID_VOXEL ? by_channels<LP_GRID_VOXEL>(tgt, m, rays, sp, n_cu, stream)
                                     : by_channels<LP_GRID_TRIPLANE>(tgt, m, rays, sp, n_cu, stream);
}

}  // namespace lp
