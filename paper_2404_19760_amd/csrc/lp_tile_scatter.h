// Scatter of a 32-sample step into a structure, one atomic add per texel and channel that the step touches: the
// gradient of the Renderer's backward (tile kernels) and what the Splatter pushes.  A step is a tile (four
// neighbouring rays, eight samples of each: column 8 i + k is sample k of ray i) or 32 samples of one ray.
#pragma once
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_mfma_bwd_common.h"
#include "lp_splat_common.h"
#include "lp_tile_lds.h"

namespace lp {

namespace {

constexpr int kTileRays = 4;                     // rays of a tile
constexpr int kTileSamples = 32 / kTileRays;     // samples of each per step

// What is scattered.
//   kGradient  a feature gradient per sample
//   kPushRay   the Splatter: one vector for all samples of a ray, and the weights themselves into a structure of one
//              channel; weights with complements from the fp64 index, as the result is divided by their sums; samples
//              that do not exist (past a ray's end) push nothing
//   kPushPoints  the Splatter with an MLP: the same with a vector per sample
enum class Scatter { kGradient, kPushRay, kPushPoints };

// ---- a step as a matrix product ----
// The samples of a step lie in a small window of texels (of each plane).  The window's gradient is
//     window[texel][channel] = sum over the 32 samples of weight[texel][sample] * dF[sample][channel],
// a contraction over the samples that the matrix cores take in fp32 (no operand splitting: the weights
// and the gradient are the same fp32 values a scalar scatter would multiply), and each texel that was
// touched gets one atomic add per channel, instead of one per run of samples in a cell and corner.
// The weight of a texel is the product of its coordinates' weights along the axes (1 - f at the sample's cell,
// f at the next, 0 elsewhere); these stand in an LDS table [axis][coordinate in the window][sample],
// from which lane = texel reads the samples of its lane group as 16-byte vectors.  Where a ray pushes one vector, the
// weights of its samples are summed first: the contraction then runs over the step's four groups of eight samples.
constexpr int kWinExtent = 12;                       // texels of a window along one axis at most
constexpr int kWinTexels = 512;                      // texels of a window of a grid at most; larger ones are split
constexpr int kWinPlaneTexels = 128;                 // the same of a plane
constexpr int kWinRow = 144;                         // bytes of a table row: 32 samples (and 16 of padding: no bank conflicts)
constexpr int kWinZeroRow = 3 * kWinExtent;          // a row of zeros, for lanes without a texel
constexpr int kWinOffsets = (kWinZeroRow + 1) * kWinRow;
constexpr int kWinMarks = kWinOffsets + 32 * 4;      // a byte per texel: touched
constexpr int kWinList = kWinMarks + kWinTexels;     // the touched texels, 16 bits each: at most 8 per sample
constexpr int kWinBytes = kWinList + 32 * 8 * 2;
static_assert(kWinBytes <= 8192 && kWinBytes % 16 == 0 && kWinOffsets % 16 == 0, "the table fits a wave's area");

struct Window {
    int lo[3], ext[3];   // uniform: first texel and number of texels along each axis
};

// Windows for the steps of a single ray: the naive Splatter's take the walk (without neighbours there is little to merge); those of
// the Splatter with an MLP a window if the whole step fits one (384 and 1600 rays over structures of 24 texels an axis, push: 1.1
// to 2 times as fast as the walk; split windows over 160 an axis 0.9 to 1.05 times, their prior's gradient 0.89 to 0.99); the
// Renderer's also several.
enum class RayWindows { kNone, kWhole, kSplit };

// v of another lane of the row of 16 (a permutation: every lane has a source)
template <int CTRL>
__device__ __forceinline__ int row_perm(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}

// extremes over the members among lanes 0 .. 31 (both lane groups hold the same cells; one member at least)
__device__ __forceinline__ Window find_window(const Cell3& c, bool member)
{
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = member ? c.i[a] : 0x7fffffff;
        hi[a] = member ? c.i[a] : 0;
    }
    auto step = [&](auto perm) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = min(lo[a], perm(lo[a]));
            hi[a] = max(hi[a], perm(hi[a]));
        }
    };
    step([](int v) { return row_perm<0xb1>(v); });    // lane ^ 1
    step([](int v) { return row_perm<0x4e>(v); });    // lane ^ 2
    step([](int v) { return row_perm<0x141>(v); });   // mirrored halves of a row
    step([](int v) { return row_perm<0x140>(v); });   // mirrored row
    Window w;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        w.lo[a] = min(__builtin_amdgcn_readlane(lo[a], 0), __builtin_amdgcn_readlane(lo[a], 16));
        w.ext[a] = max(__builtin_amdgcn_readlane(hi[a], 0), __builtin_amdgcn_readlane(hi[a], 16)) - w.lo[a] + 2;
    }
    return w;
}

template <int KIND>
__device__ __forceinline__ bool window_fits(const Window& w)
{
    if (max(w.ext[0], max(w.ext[1], w.ext[2])) > kWinExtent) return false;
    if constexpr (KIND == LP_GRID_TRIPLANE)
        return max(w.ext[0] * w.ext[1], max(w.ext[1] * w.ext[2], w.ext[2] * w.ext[0])) <= kWinPlaneTexels;
    else
        return w.ext[0] * w.ext[1] * w.ext[2] <= kWinTexels;
}

// n / d for 0 <= n < 2^12 and the reciprocal inv of d <= 144 (the offset of one half keeps the rounding away)
__device__ __forceinline__ int small_div(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }

// dFt: feature gradient, lane = channel (16 channels: lanes 16 .. 31 repeat lanes 0 .. 15), register r =
// column d_row(r, grp) of the step.  `member`: the lane's sample belongs to the window (others have weight
// zero).  `area`: the wave's LDS area for the table.  `sums`: the Splatter's weight sums.
template <int KIND, int C, Scatter WHAT>
__device__ __forceinline__ void scatter_window(const GridDev& g, float* const d_grid[3], float* const* sums, int scene,
                                               uint32_t area, const Window& win, const Cell3& cell, bool member,
                                               const f32x16& dFt, int lane)
{
    constexpr bool kPushes = WHAT != Scatter::kGradient, kOfRay = WHAT == Scatter::kPushRay;
    const int col = lane & 31, grp = lane >> 5;
    // the table: zeros, then this sample's two entries per axis (lane group 0 the lower, 1 the upper)
    wave_lds_fence();
    for (int i = lane; i < (kWinZeroRow + 1) * kWinRow / 16; i += 64)
        lds_put<u32x4>(area + 16 * i, u32x4{0u, 0u, 0u, 0u});
    wave_lds_fence();
    const int pos = slot_to_sample(col);   // 16 grp + r for column d_row(r, grp)
    if (member) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int row = a * kWinExtent + cell.i[a] - win.lo[a] + grp;
            lds_put<float>(area + row * kWinRow + pos * 4, grp ? cell.f[a] : kPushes ? cell.g[a] : 1.0f - cell.f[a]);
        }
    }
    wave_lds_fence();

    constexpr int kLanes = C == 32 ? 32 : 16;         // texels per matrix product
    constexpr int kVec = C == 32 ? 4 : 2;             // 16-byte vectors of samples per lane
    const int slot = lane & (kLanes - 1);
    const int first = C == 32 ? 64 * grp : 32 * (lane >> 4);   // byte offset of this lane's samples in a row
    float b16[8];
    if constexpr (C == 16) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float a = dFt[k], b = dFt[k + 8];
            asm("" : "+v"(a), "+v"(b));   // (or the compiler turns the choice into an indexed read of dFt)
            b16[k] = (lane & 16) ? b : a;
        }
    }

    constexpr int kPlanes = KIND == LP_GRID_TRIPLANE ? 3 : 1;
#pragma unroll
    for (int pl = 0; pl < kPlanes; ++pl) {
        // axes of the window, slowest first
        const int a0 = KIND == LP_GRID_TRIPLANE ? pl : 0, a1 = KIND == LP_GRID_TRIPLANE ? (pl + 1) % 3 : 1;
        const int e1 = win.ext[a1], e2 = KIND == LP_GRID_TRIPLANE ? 1 : win.ext[2];
        const int total = win.ext[a0] * e1 * e2;
        // A large window is mostly empty: the samples of a step lie along a line through it. Its products then run over
        // the texels that a sample reaches, in the order of the window (a product over 32 texels of 32 channels occupies
        // the matrix cores for 1024 cycles; finding the texels takes some 400).  Windows up to two products stay whole: at
        // most one product is to be saved there.  Hash table over a 128^3 lattice, 5.6 -> 3.4 products a step: backward
        // 0.457 -> 0.412 ms; 5003 rays in random order through 97 x 128 x 75 x 16 voxels, whose steps of one ray fit one
        // window of 512 texels instead of several of 128: 0.319 -> 0.268 ms.
        int n_texels = total;
        const bool listed = KIND != LP_GRID_TRIPLANE && total > 2 * kLanes;
        if (listed) {
            lds_put<u32x2>(area + kWinMarks + 8 * lane, u32x2{0u, 0u});
            wave_lds_fence();
            if (member) {   // the lane group's face of the sample's cell
                const uint32_t at = area + kWinMarks + ((cell.i[0] - win.lo[0] + grp) * e1 + cell.i[1] - win.lo[1]) * e2 +
                                    cell.i[2] - win.lo[2];
                const uint8_t one = 1;
                lds_put<uint8_t>(at, one);
                lds_put<uint8_t>(at + 1, one);
                lds_put<uint8_t>(at + e2, one);
                lds_put<uint8_t>(at + e2 + 1, one);
            }
            wave_lds_fence();
            n_texels = 0;
            for (int n = 0; n < total; n += 64) {
                const bool touched = lds_get<uint8_t>(area + kWinMarks + n + lane) != 0;
                const unsigned long long all = __ballot(touched);
                const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)all, 0u));
                if (touched) lds_put<uint16_t>(area + kWinList + 2 * (n_texels + before), (uint16_t)(n + lane));
                n_texels += __popcll(all);
            }
            wave_lds_fence();
        }
        const float inv12 = __builtin_amdgcn_rcpf((float)(e1 * e2)), inv2 = __builtin_amdgcn_rcpf((float)e2);
        size_t scene_at;   // first texel of the scene
        if constexpr (KIND == LP_GRID_TRIPLANE) scene_at = (size_t)scene * g.N[a0] * g.N[a1];
        else if constexpr (KIND == LP_GRID_HASH) scene_at = (size_t)scene * g.hash_size;
        else scene_at = (size_t)scene * g.N[0] * g.N[1] * g.N[2];
        char* out = reinterpret_cast<char*>(d_grid[pl] + scene_at * C);
        for (int n0 = 0; n0 < n_texels; n0 += kLanes) {
            const bool live = n0 + slot < n_texels;
            const int at = live ? n0 + slot : 0, n = listed ? (int)lds_get<uint16_t>(area + kWinList + 2 * at) : at;   // (lanes without a texel: weights zero, the first one's address)
            const int t0 = small_div(n, inv12), rest = n - t0 * (e1 * e2);
            const int t1 = KIND == LP_GRID_TRIPLANE ? rest : small_div(rest, inv2), t2 = rest - t1 * e2;
            unsigned off;
            if constexpr (KIND == LP_GRID_TRIPLANE)
                off = ((unsigned)(win.lo[a0] + t0) * (unsigned)g.N[a1] + (unsigned)(win.lo[a1] + t1)) * C;
            else if constexpr (KIND == LP_GRID_HASH)   // (a table whose size is a power of two; colliding texels add up)
                off = (((unsigned)(win.lo[0] + t0) ^ (unsigned)(win.lo[1] + t1) * 2654435761u ^
                        (unsigned)(win.lo[2] + t2) * 805459861u) & (g.hash_size - 1u)) * C;
            else
                off = (((unsigned)(win.lo[0] + t0) * (unsigned)g.N[1] + (unsigned)(win.lo[1] + t1)) * (unsigned)g.N[2] +
                       (unsigned)(win.lo[2] + t2)) * C;
            const uint32_t r0 = area + (live ? a0 * kWinExtent + t0 : kWinZeroRow) * kWinRow + first;
            const uint32_t r1 = area + (live ? a1 * kWinExtent + t1 : kWinZeroRow) * kWinRow + first;
            const uint32_t r2 = area + (live ? 2 * kWinExtent + t2 : kWinZeroRow) * kWinRow + first;
            float w[4 * kVec];
#pragma unroll
            for (int v = 0; v < kVec; ++v) {
                const f32x4 x = lds_get<f32x4>(r0 + 16 * v), y = lds_get<f32x4>(r1 + 16 * v);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[4 * v + e] = x[e] * y[e];
                if constexpr (KIND != LP_GRID_TRIPLANE) {
                    const f32x4 z = lds_get<f32x4>(r2 + 16 * v);
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[4 * v + e] *= z[e];
                }
            }
            if constexpr (kPushes) {
                float sum = 0.0f;
#pragma unroll
                for (int k = 0; k < 4 * kVec; ++k) sum += w[k];
                if constexpr (C == 16) sum += __shfl_xor(sum, 16, 64);
                sum += __shfl_xor(sum, 32, 64);
                if (lane < kLanes && live && sum != 0.0f) atomicAdd(sums[pl] + scene_at + off / C, sum);
            }
            if constexpr (kOfRay) {
#pragma unroll
                for (int v = 0; v < kVec; ++v) w[v] = (w[4 * v] + w[4 * v + 1]) + (w[4 * v + 2] + w[4 * v + 3]);
            }
            // offsets of all texels of this product, for the lanes that will hold their rows
            wave_lds_fence();
            if (lane < kLanes) lds_put<uint32_t>(area + kWinOffsets + 4 * slot, off);
            wave_lds_fence();
            auto add = [&](unsigned texel_off, float v) {
                if (v != 0.0f) atomicAdd(reinterpret_cast<float*>(out + 4u * (texel_off + (unsigned)(lane & (C - 1)))), v);
            };
            if constexpr (C == 32) {
                f32x16 acc = zero16();
#pragma unroll
                for (int r = 0; r < (kOfRay ? 4 : 16); ++r)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[r], dFt[kOfRay ? 4 * r : r], acc, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (n0 + 8 * q >= n_texels) break;
                    const u32x4 o = lds_get<u32x4>(area + kWinOffsets + 4 * (8 * q + 4 * grp));
#pragma unroll
                    for (int p = 0; p < 4; ++p) add(o[p], acc[4 * q + p]);
                }
            } else {
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < (kOfRay ? 2 : 8); ++k)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[k], b16[kOfRay ? 4 * k : k], acc, 0, 0, 0);
                const u32x4 o = lds_get<u32x4>(area + kWinOffsets + 16 * (lane >> 4));
#pragma unroll
                for (int p = 0; p < 4; ++p) add(o[p], acc[p]);
            }
        }
    }
}

// The walk on a step of the tile kernel: records and feature gradient go through LDS in the order of the
// walk (16 positions per lane group): samples of one ray in order, or ray after ray of a tile, every other
// one backwards, so that the step from ray to ray is a short one.
template <int KIND, int C, Scatter WHAT>
__device__ __forceinline__ void scatter_walk(const GridDev& g, float* const d_grid[3], float* const* sums, int scene, char* area,
                                             const Cell3& cell, bool valid, const f32x16& dFt, int lane, bool tile)
{
    constexpr bool kPushes = WHAT != Scatter::kGradient, kOfRay = WHAT == Scatter::kPushRay;
    const int col = lane & 31, grp = lane >> 5;
    auto flip = [tile](int c) { return (tile && (c & 8)) ? c ^ 7 : c; };   // column <-> position of the walk
    float* info = reinterpret_cast<float*>(area);
    float* grad = reinterpret_cast<float*>(area + 2048);
    wave_lds_fence();
    if (grp == 0) {
        float* rec = info + flip(col) * 16;
        write_scatter_record<KIND, C, kPushes>(rec, g, cell);
        if (kPushes && !valid) {
#pragma unroll
            for (int i = 0; i < (KIND == LP_GRID_TRIPLANE ? 12 : 8); ++i) rec[i] = 0.0f;
        }
    }
    if (!kOfRay && col < C) {
#pragma unroll
        for (int r = 0; r < 16; ++r) grad[flip(d_row(r, grp)) * C + col] = dFt[r];
    }
    wave_lds_fence();
    f32x16 v;
    [[maybe_unused]] const unsigned there = (unsigned)__ballot(valid);   // a bit per column
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if constexpr (kOfRay) v[r] = grp ? dFt[8 + 4 * (r / 8)] : dFt[4 * (r / 8)];   // position 16 grp + r: ray 2 grp + r / 8
        else v[r] = grad[(16 * grp + r) * C + (col & (C - 1))];
        // what does not exist pushes nothing: weight zero alone would turn an infinite feature into an undefined one
        if constexpr (kPushes) v[r] = ((there >> flip(16 * grp + r)) & 1u) ? v[r] : 0.0f;
    }
    scatter_channels<KIND, C, true>(g, d_grid, scene, info, v, col, grp);
    if constexpr (kPushes) scatter_weights<KIND, C, true>(g, sums, scene, info, col, grp);
    wave_lds_fence();
}

// A step's scatter.  Where the samples of the whole step spread too far for one window, they are taken as two or four
// runs of consecutive samples (of every ray of the tile) with a window each: rays that leave the unit cube of contract
// coordinates between two samples, mostly.  The products would spread an infinite or
// undefined gradient over its window, so a step that holds one takes the walk, which keeps it to the sample's own corners.
// Steps of a single ray: see RayWindows; `windows` false: the walk.
template <int KIND, int C, Scatter WHAT = Scatter::kGradient, RayWindows RAYS = WHAT == Scatter::kGradient ? RayWindows::kSplit : RayWindows::kNone>
__device__ __forceinline__ void scatter_step(const GridDev& g, float* const d_grid[3], int scene, uint32_t area,
                                             char* area_ptr, const Cell3& cell, const f32x16& dFt, int lane, bool tile,
                                             float* const* sums = nullptr, bool valid = true, bool windows = true)
{
    constexpr bool kOfRay = WHAT == Scatter::kPushRay;
    const int col = lane & 31, k = tile ? (col & (kTileSamples - 1)) : col, full = tile ? kTileSamples : 32;
    float probe = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (!kOfRay || r % 4 == 0) probe = fmaf(dFt[r], 0.0f, probe);
    const bool finite = __ballot(probe != 0.0f) == 0ull && (RAYS != RayWindows::kNone || tile) && windows;
    int len = full;
    Window win;
    bool fits = false;
    if (finite) {
        win = find_window(cell, true);
        fits = window_fits<KIND>(win);
    }
    while (!fits && finite && len > full / 4 && (RAYS == RayWindows::kSplit || tile)) {
        len >>= 1;
        fits = true;
        for (int p = full - len; p >= 0 && fits; p -= len) {
            win = find_window(cell, (unsigned)(k - p) < (unsigned)len);
            fits = window_fits<KIND>(win);
        }
    }
    if (!fits) {
        scatter_walk<KIND, C, WHAT>(g, d_grid, sums, scene, area_ptr, cell, valid, dFt, lane, tile);
        return;
    }
    for (int p = 0;;) {   // `win` is the first run's
        scatter_window<KIND, C, WHAT>(g, d_grid, sums, scene, area, win, cell, valid && (unsigned)(k - p) < (unsigned)len,
                                      dFt, lane);
        p += len;
        if (p >= full) break;
        win = find_window(cell, (unsigned)(k - p) < (unsigned)len);
    }
}

// The Splatter's work items: tiles of consecutive rays or single rays, `waves_per_group` of them to a group, the groups in
// a scrambled order.
struct PushOrder {
    long long n_groups, group_mul;
    int tiles;
};

// Tiles where the longest wave has at most twice as many steps that way: a tile's step is cheaper, but a launch of few rays
// spreads over more waves ray by ray.  Push time in single rays over that in tiles, neighbouring rays, for 16- and
// 32-channel voxel grids, a triplane and a hash table at 64 and 160 samples: 2.0 .. 4.7 where the steps are as many,
// 1.7 .. 4.4 at 1.33 times as many, 1.08 .. 3.5 at twice, 0.95 .. 2.8 at four times (160^3 x 32 voxels, whose adds bind
// either way, at 1.0).  With an MLP, 48^2 and 64^2 pixels (twice the steps) up to one texel apart: forward 1.0 .. 2.4.
inline PushOrder push_order(const RaysDev& rays, long long waves, int waves_per_group, double tiles_up_to = 2.0)
{
    auto rounds = [&](long long items) { return (items + waves - 1) / waves; };
    const long long n_tiles = (rays.M + kTileRays - 1) / kTileRays;
    const long long tile_steps = rounds(n_tiles) * ((rays.S + kTileSamples - 1) / kTileSamples);
    const long long ray_steps = rounds(rays.M) * ((rays.S + 31) / 32);
    PushOrder o;
    o.tiles = (double)tile_steps <= tiles_up_to * (double)ray_steps;
    const long long items = o.tiles ? n_tiles : rays.M;
    o.n_groups = (items + waves_per_group - 1) / waves_per_group;
    o.group_mul = splat_group_multiplier(o.n_groups);
    return o;
}

// Splatter with an MLP: cells between the rays of a tile.  (64^2 pixels over 160^3 voxels, 1.3 voxels from pixel to pixel: push
// 1.09 ms with 3, where most rays go one by one, 0.79 with 6, 0.76 with 9.  Pixels two texels apart are tiles with 9 and gain, 1.0 .. 2.0
// from 64^2 pixels x 64 points on; those three apart are none, and gain by neither.)
constexpr int kPushApart = 9;

// Whether the rays run in tiles: in three of four among 64 tiles they lie side by side, within `near_by` texels at both ends, and a step is
// at most `step` texels long in the middle.  All threads of a workgroup call it, and every workgroup and the other kernel of a pair
// find the same: no contraction of products and sums.  (One wave looks, in fp32 and with all loads under way at once: every launch
// waits for it.)
__device__ __forceinline__ bool rays_run_in_tiles(const GridDev& g, const RaysDev& rays, float near_by, float step)
{
#pragma clang fp contract(off)
    __shared__ int together;
    if (threadIdx.x < 64) {
        const long long n_tiles = (rays.M + kTileRays - 1) / kTileRays;
        const long long first = (long long)threadIdx.x * n_tiles / 64 * kTileRays;
        float near[kTileRays], far[kTileRays], o[kTileRays][3], d[kTileRays][3];
#pragma unroll
        for (int i = 0; i < kTileRays; ++i) {
            const long long r = min(first + i, rays.M - 1);
            near[i] = rays.near[r];
            far[i] = rays.far[r];
#pragma unroll
            for (int a = 0; a < 3; ++a) { o[i][a] = rays.origins[3 * r + a]; d[i][a] = rays.dirs[3 * r + a]; }
        }
        const float contract = (float)g.contract;
        auto texel = [&](int i, int a, float t) {
#pragma clang fp contract(off)
            float x = o[i][a] + t * d[i][a];
            if (contract > 0.0f) {
                const float m = fabsf(x), far = 0.5f * ((2.0f - contract) * (1.0f - 1.0f / fmaxf(m, 1.0f)) + contract);
                x = m <= 1.0f ? 0.5f * contract * x : x < 0.0f ? -far : far;
            }
            return fminf(fmaxf((x - (float)g.amin[a]) * (float)g.scale[a], 0.0f), (float)(g.N[a] - 1));
        };
        const float middle = 0.5f * (near[0] + far[0]), ahead = middle + (float)kTileSamples * (far[0] - near[0]) / (float)rays.S;
        bool apart = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float n0 = texel(0, a, near[0]), f0 = texel(0, a, far[0]);
#pragma unroll
            for (int i = 1; i < kTileRays; ++i)
                apart = apart || !(fabsf(texel(i, a, near[i]) - n0) <= near_by) || !(fabsf(texel(i, a, far[i]) - f0) <= near_by);
            apart = apart || !(fabsf(texel(0, a, ahead) - texel(0, a, middle)) <= step);
        }
        const int n = __popcll(__ballot(!apart));
        if (threadIdx.x == 0) together = n;
    }
    __syncthreads();
    return 4 * together >= 3 * 64;
}

// Whether the four rays from `first` on (those below `end`) run side by side: in one scene, and within APART cells of the
// first at both ends.
template <int APART = 3, class CellOf>
__device__ __forceinline__ bool side_by_side(const RaysDev& rays, long long first, long long end, int col, CellOf cell_of)
{
    const RayGeom q = load_ray_geom(rays, min(first + col / kTileSamples, end - 1));
    const Cell3 c0 = cell_of(q, 0), c1 = cell_of(q, rays.S - 1);
    bool apart = q.scene != __builtin_amdgcn_readfirstlane(q.scene);
#pragma unroll
    for (int a = 0; a < 3; ++a)
        apart = apart || abs(c0.i[a] - __builtin_amdgcn_readfirstlane(c0.i[a])) > APART ||
                abs(c1.i[a] - __builtin_amdgcn_readfirstlane(c1.i[a])) > APART;
    return __ballot(apart) == 0ull;
}

}  // namespace

}  // namespace lp
