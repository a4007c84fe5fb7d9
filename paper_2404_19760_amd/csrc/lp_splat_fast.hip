// Naive Splatter forward (Section 3.3 "Splatter": every point of a pixel's ray pushes the pixel's
// feature vector into the cell that contains it).
//
// What bounds it: the rate of atomic adds (2.1e10 64-byte lines/s on this chip). Pushed ray by ray, a point adds
// about 10 lines after runs in a cell are merged. Neighbouring rays reach the same texels, so a step takes several of them and
// adds once per texel what a matrix product of interpolation weights and pixel features gives:
//   - images: patches of 8 x 4 pixels, eight points of each (lp_splat_patch.h), 1.55 lines per point, weight sums included;
//   - other lists of rays: tiles of four neighbouring ones (lp_tile_scatter.h), 3.93 lines per point on the same rays; rays that
//     do not run side by side one after the other, 32 points per step, by the run-merging walk.
// 160^3 x 32 voxels, 4 x 128^2 rays x 160 points: 5.41 ms ray by ray, 2.18 in tiles (4.12e7 atomic requests of the L2: 90 % of
// the rate of the adds), 1.00 in patches (1.62e7: 77 %; one wave per SIMD, whose LDS holds the weights).
// Items are visited in scrambled order like the Renderer's backward
// (atomic adds of neighbouring rays queue up at the same L2 channel).
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_mfma_bwd_common.h"
#include "lp_splat_common.h"
#include "lp_splat_patch.h"
#include "lp_tile_scatter.h"

#include <algorithm>

namespace lp {

namespace {

constexpr int kWaves = 4;
constexpr int kPatchRays = 32;    // of a patch: see lp_splat_patch.h
using Patch = PatchLds<kPatchRays>;
constexpr int kArea = kWinBytes;   // LDS of a wave: the window's table, or the records of a walk
static_assert(kArea <= Patch::kBytes && kWaves * Patch::kBytes <= 160 * 1024, "LDS of a patch's wave");
static_assert(kArea >= 32 * 16 * 4, "the walk's records");

// Pushes the rays [first, end) (four at most), points j_from .. j_to - 1: as a tile if `tiles` and they run side by side,
// else one after the other.
template <int KIND, int C, bool CC>
__device__ __forceinline__ void push_rays(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, long long first, long long end,
                                          int j_from, int j_to, bool tiles, char* area_ptr, int lane)
{
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)area_ptr;
    const int col = lane & 31;
    const bool tile = tiles && side_by_side(rays, min(first + col / kTileSamples, end - 1), [&](const RayGeom& r, int j) { return sample_cell<CC>(tgt, r, j); });
    const int n_sub = tile ? 1 : (int)(end - first);
    for (int sub = 0; sub < n_sub; ++sub) {
        const long long r = first + (tile ? col / kTileSamples : sub);
        const bool ray_ok = r < end;
        const RayGeom q = load_ray_geom(rays, min(r, end - 1));
        const int scene = __builtin_amdgcn_readfirstlane(q.scene);
        // the pixels' features of this lane's channel (16 channels: both halves of a lane group)
        f32x16 val;
#pragma unroll
        for (int i = 0; i < kTileRays; ++i) {
            const long long at = min(first + (tile ? i : sub), end - 1);
            const float v = sp.feats[(size_t)at * C + (col & (C - 1))];
#pragma unroll
            for (int e = 0; e < 4; ++e) val[4 * i + e] = v;
        }
        const int step = tile ? kTileSamples : 32, k = tile ? col % kTileSamples : col;
        for (int j0 = j_from; j0 < j_to; j0 += step) {
            const int j = j0 + k;
            const Cell3 c = sample_cell<CC>(tgt, q, min(j, rays.S - 1));
            uint32_t lane_here = lane;   // (or what the scatter derives from the lane number is kept through the loop)
            refresh(lane_here);
            scatter_step<KIND, C, Scatter::kPushRay>(tgt, sp.theta, scene, area, area_ptr, c, val, lane_here, step,
                                                     sp.theta_w, ray_ok && j < j_to);
        }
    }
}

// Patches are taken from this many rays on, where neighbouring pixels are close enough: 160^3 voxels (16 and 32 channels, 24 and 160
// points a ray), push time in tiles of a row over that in patches: 1.3 .. 1.5 at 0.66 texels from pixel to pixel, 2.1 .. 3.2 at
// 0.2 and 0.33, 0.25 .. 0.9 at 1.3 (a step then takes one point at a time). 160^2 triplanes 1.2 .. 5.6 at 1.3, 0.45 .. 1.75 at
// 2.1.  Over structures of 24 and 64 texels an axis: 384 rays 0.04 .. 1.5, 1600 rays 0.75 .. 3.6, 3072 rays 1.7 .. 6.4.
// What is no image pays for the question, from 2048 rays on: lists 2 to 4 us for the second launch (3072 rays x 24 points, 80 to
// 210 us: 0.97 .. 0.98 of the speed without it), images whose pixels are too far apart 4 to 8 us (2112 rays, 80 to 640 us:
// 0.92 .. 0.99, the slowest at 1.0 to 1.2 texels a pixel, where a row is looked for and found).
constexpr long long kMinRays = 2048;
template <int KIND>
__device__ __forceinline__ long long image_row(const GridDev& g, const RaysDev& rays)
{
    __shared__ int found;
    return find_row(g, rays, KIND == LP_GRID_TRIPLANE ? 1.5 : 0.9, 1e30, found);
}

// Rays in their order.  PATCHES: the patch kernel has been launched before and takes what it finds to be an image (an
// instantiation of its own: launches of few rays, which never look for one, took 1 us of 40 longer with the search in their code).
template <int KIND, int C, bool CC, bool PATCHES>
__global__ __launch_bounds__(kWaves * 64, 3) void splat_naive_kernel(GridDev tgt, RaysDev rays, SplatDev sp, PushOrder order)
{
    __shared__ __align__(16) char areas[kWaves][kArea];
    if constexpr (PATCHES) {
        if (image_row<KIND>(tgt, rays) != 0) return;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rays_per_item = order.tiles ? kTileRays : 1;
    const RaySchedule sched = ray_schedule(order.n_groups * kWaves, kWaves);
    for (long long seq = sched.first; seq < sched.end; seq += sched.stride) {
        const long long first = (((seq / kWaves) * order.group_mul % order.n_groups) * kWaves + seq % kWaves) * rays_per_item;
        if (first >= rays.M) continue;
        push_rays<KIND, C, CC>(tgt, rays, sp, first, min(first + rays_per_item, rays.M), 0, rays.S, order.tiles != 0, areas[wave], lane);
    }
}

// Points [from, from + len) of a step of a patch into plane `pl`, of all rays or (`only` >= 0) of one.  false: they reach too
// many texels (nothing is pushed).  The push is the product weights[texel][ray] x feature[ray][channel], in fp32.
template <int KIND, int C>
__device__ __forceinline__ bool push_points(const GridDev& g, const SplatDev& sp, int scene, uint32_t area, const PatchCells& cells,
                                            int from, int len, int only, int pl, const float (&val)[C / 2], int lane)
{
    constexpr int kLanes = C == 32 ? 32 : 16;          // texels of a product
    constexpr int kRays = C == 32 ? 16 : 8;            // of a lane
    const int n_slots = patch_weights<KIND, C, kPatchRays>(area, g, cells, from, len, only, pl, lane);
    if (n_slots <= 0) return n_slots == 0;
    const size_t scene_at = scene_texel<KIND>(g, pl, scene);
    char* out = reinterpret_cast<char*>(sp.theta[pl] + scene_at * C);
    const int slot = lane & (kLanes - 1), part = lane / kLanes;
    for (int n0 = 0; n0 < n_slots; n0 += kLanes) {
        const bool live = n0 + slot < n_slots;
        const int at = live ? n0 + slot : n0;
        float w[kRays], sum = 0.0f;
#pragma unroll
        for (int v = 0; v < kRays / 4; ++v) {
            const f32x4 x = lds_get<f32x4>(area + at * Patch::kRow + part * kRays * 4 + 16 * v);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[4 * v + e] = live ? x[e] : 0.0f;
                sum += w[4 * v + e];
            }
        }
        if constexpr (C == 16) sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        if (lane < kLanes && live && sum != 0.0f)
            atomicAdd(sp.theta_w[pl] + scene_at + lds_get<uint32_t>(area + Patch::OFFSETS + 4 * at) / C, sum);
        auto add = [&](unsigned texel_off, float v) {
            if (v != 0.0f) atomicAdd(reinterpret_cast<float*>(out + 4u * (texel_off + (unsigned)(lane & (C - 1)))), v);
        };
        if constexpr (C == 32) {
            f32x16 acc = zero16();
#pragma unroll
            for (int r = 0; r < kRays; ++r) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[r], val[r], acc, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {   // (slots that do not exist: sums of zeros, nothing is added)
                const u32x4 o = lds_get<u32x4>(area + Patch::OFFSETS + 4 * (n0 + 8 * q + 4 * part));
#pragma unroll
                for (int p = 0; p < 4; ++p) add(o[p], acc[4 * q + p]);
            }
        } else {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int r = 0; r < kRays; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], val[r], acc, 0, 0, 0);
            const u32x4 o = lds_get<u32x4>(area + Patch::OFFSETS + 4 * (n0 + 4 * part));
#pragma unroll
            for (int p = 0; p < 4; ++p) add(o[p], acc[p]);
        }
    }
    return true;
}

// Images, patch after patch (lp_splat_patch.h).  An item is a patch and `seg` points of its rays.  Where rays of a line are not
// neighbours or not finite, they are pushed line by line like a list's.
template <int KIND, int C, bool CC>
__global__ __launch_bounds__(kWaves * 64) void splat_patch_kernel(GridDev tgt, RaysDev rays, SplatDev sp, int seg)
{
    extern __shared__ uint4 lds_raw[];
    const long long row = image_row<KIND>(tgt, rays);
    if (row == 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const area_ptr = reinterpret_cast<char*>(lds_raw) + wave * Patch::kBytes;
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)area_ptr;
    constexpr int kPlanes = KIND == LP_GRID_TRIPLANE ? 3 : 1;
    const PatchGrid<kPatchRays> grid(rays.M, row);
    const int S = rays.S;
    const long long n_segs = (S + seg - 1) / seg, n_items = grid.count * n_segs;
    const long long n_groups = (n_items + kWaves - 1) / kWaves;
    const long long mul = n_groups % 7919 ? 7919 : n_groups % 7907 ? 7907 : 1;   // scrambled order: a prime that does not divide their number
    const RaySchedule sched = ray_schedule(n_groups * kWaves, kWaves);
    for (long long seq = sched.first; seq < sched.end; seq += sched.stride) {
        const long long item = (seq / kWaves) * mul % n_groups * kWaves + seq % kWaves;
        if (item >= n_items) continue;
        const long long patch = item % grid.count;
        const int j_from = (int)(item / grid.count) * seg, j_to = min(j_from + seg, S);
        bool there;
        const RayGeom q = load_ray_geom(rays, grid.ray(patch, lane & (kPatchRays - 1), there));
        // features: matrix operand, lane = channel, register r = ray kRays (lane / C) + r
        constexpr int kRays = C / 2;
        float val[kRays], probe = 0.0f;
#pragma unroll
        for (int r = 0; r < kRays; ++r) {
            bool has;
            const long long at = grid.ray(patch, kRays * (lane / C) + r, has);
            val[r] = has ? sp.feats[(size_t)at * C + (lane & (C - 1))] : 0.0f;
            probe = fmaf(val[r], 0.0f, probe);   // (an infinite feature would spread over the window)
        }
        const bool finite = __ballot(probe != 0.0f) == 0ull;
        patch_parts(patch_lines<kPatchRays, CC>(tgt, q, there, S, lane), [&](int y0, int y1, bool by_lines) {
            const int y = (lane & (kPatchRays - 1)) / PatchGrid<kPatchRays>::kW;
            const bool ok = there && y >= y0 && y < y1;
            const unsigned long long oks = __ballot(ok);
            if (oks == 0ull) return;
            if (by_lines || !finite) {
                for (int t = 2 * y0; t < 2 * y1; ++t) {
                    long long first, end;
                    grid.line(patch, t / 2, first, end);
                    first += (t & 1) * kTileRays;
                    end = min(end, first + kTileRays);
                    if (first < end) push_rays<KIND, C, CC>(tgt, rays, sp, first, end, j_from, j_to, true, area_ptr, lane);
                }
                return;
            }
            const int scene = __builtin_amdgcn_readfirstlane(__shfl(q.scene, __builtin_ctzll(oks), 64));
            for (int j0 = j_from; j0 < j_to; j0 += kPatchPoints) {
                const PatchCells cells = patch_cells<CC>(tgt, q, ok, j0, j_to, S);
#pragma unroll 1
                for (int pl = 0; pl < kPlanes; ++pl)
                    patch_steps<kPatchRays>([&](int from, int len, int only) {
                        return push_points<KIND, C>(tgt, sp, scene, area, cells, from, len, only, pl, val, lane);
                    });
            }
        });
    }
}

template <int KIND, int C, bool CC>
hipError_t launch(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    const bool patches = rays.M >= kMinRays;
    if (patches) {
        auto kernel = splat_patch_kernel<KIND, C, CC>;
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kWaves * Patch::kBytes);
        if (e != hipSuccess) return e;
        const long long blocks = (n_cu + 7) / 8 * 8, waves = blocks * kWaves;
        // about eight items for every wave, of a step at least
        const long long points = (rays.M / kPatchRays + 1) * rays.S / (8 * waves);
        const int seg = (int)std::min<long long>(std::max<long long>(points / kPatchPoints * kPatchPoints, kPatchPoints), rays.S);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kWaves * 64), kWaves * Patch::kBytes, stream, tgt, rays, sp, seg);
    }
    long long blocks = 4LL * n_cu;   // four workgroups per compute unit
    blocks = (blocks + 7) / 8 * 8;
    const PushOrder order = push_order(rays, blocks * kWaves, kWaves);
    if (blocks > order.n_groups) blocks = (order.n_groups + 7) / 8 * 8;
    auto kernel = patches ? splat_naive_kernel<KIND, C, CC, true> : splat_naive_kernel<KIND, C, CC, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kWaves * 64), 0, stream, tgt, rays, sp, order);
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
