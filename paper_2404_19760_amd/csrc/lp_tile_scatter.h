// Scatter of a 32-sample step into a structure, one atomic add per texel and channel that the step touches: the
// gradient of the Renderer's backward (tile kernels) and what the Splatter pushes.  A step is 32
// samples: of a patch (four neighbouring pixels each of two rows, four samples of each), of a tile (four neighbouring rays, eight samples of
// each) or of one ray; with `full` samples of a ray in the step column full i + k is sample k of ray i.
#pragma once
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_mfma_bwd_common.h"
#include "lp_splat_common.h"
#include "lp_tile_lds.h"

#include <type_traits>

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
constexpr int kWinRows = 3 * kWinExtent + 1;         // rows of the table at most: the axes' one after the other, then one of zeros

// The wave's area: the table, a byte per texel of the window (of each plane) that says whether a sample reaches it, and the
// list of those that one does: where the texel is added to, and its rows of the table.
// FAR: the list holds texels of planes in different tensors (8-byte addresses, else element offsets in a scene).
template <bool FLAT, bool FAR>
struct WinLds {
    static constexpr int kMarks = FLAT ? 3 * kWinPlaneTexels : kWinTexels;
    static constexpr int kList = FAR ? 240 : 256;    // (of a grid 8 per sample at most; of planes: see scatter_window)
    static constexpr int kWhere = FAR ? 8 : 4, kWhich = FLAT ? 2 : 4;   // bytes of an entry
    static constexpr int MARKS = kWinRows * kWinRow;
    static constexpr int WHERE = MARKS + kMarks;
    static constexpr int WHICH = WHERE + kList * kWhere;
    static constexpr int kBytes = WHICH + kList * kWhich;
    static_assert(kList % 16 == 0 && kList >= kWinPlaneTexels && MARKS % 16 == 0 && WHERE % 16 == 0, "16-byte accesses; a plane's list fits");
};
constexpr int kWinBytes = 8192;
static_assert(WinLds<false, false>::kBytes <= kWinBytes && WinLds<true, false>::kBytes <= kWinBytes && WinLds<true, true>::kBytes <= kWinBytes);

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
// zero).  `area`: the wave's LDS area.  `sums`: the Splatter's weight sums.
//
// A window is mostly empty (the samples of a step lie along a line through it), and a product is the dearest thing here: the
// matrix cores take fp32 at a sixteenth of their rate in bf16.  So the products run over a list of the texels that a sample
// reaches, 16 texels each (32 channels: two products side by side), and over the texels of all three planes of a triplane
// in one list.  Against products over whole windows (32 texels of 32 channels; lists only of windows larger than two
// products; a plane at a time), backward: eight triplanes 256^2 x 32 (3.5 x 32 texels a step, now 3.8 x 16 of 55 reached) 95.5 -> 88.4 ms,
// 160^3 x 32 voxels in contract coordinates 7.0 -> 6.3, 64^3 x 32 voxels 7.3 -> 7.0, 256^3 x 16 voxels 48.2 -> 47.8 ms.
template <int KIND, int C, Scatter WHAT>
__device__ __forceinline__ void scatter_window(const GridDev& g, float* const d_grid[3], float* const* sums, int scene,
                                               uint32_t area, const Window& win, const Cell3& cell, bool member,
                                               const f32x16& dFt, int lane)
{
    constexpr bool kPushes = WHAT != Scatter::kGradient, kOfRay = WHAT == Scatter::kPushRay;
    constexpr bool kFlat = KIND == LP_GRID_TRIPLANE, kFar = kFlat && !kPushes;   // (a push keeps the planes apart: their weight sums)
    constexpr int kPlanes = kFlat ? 3 : 1;
    using L = WinLds<kFlat, kFar>;
    using Which = typename std::conditional<kFlat, uint16_t, uint32_t>::type;
    const int col = lane & 31, grp = lane >> 5;
    const int first_row[3] = {0, win.ext[0], win.ext[0] + win.ext[1]}, zero_row = first_row[2] + win.ext[2];
    // axes of the window (of plane pl), slowest first
    auto axis0 = [](int pl) { return kFlat ? pl : 0; };
    auto axis1 = [](int pl) { return kFlat ? (pl + 1) % 3 : 1; };

    // the table: zeros, then this sample's two entries per axis (lane group 0 the lower, 1 the upper), and the marks: the
    // lane group's face of the sample's cell
    wave_lds_fence();
    for (int i = lane; i < (zero_row + 1) * (kWinRow / 16); i += 64) lds_put<u32x4>(area + 16 * i, u32x4{0u, 0u, 0u, 0u});
    if (lane < L::kMarks / 16) lds_put<u32x4>(area + L::MARKS + 16 * lane, u32x4{0u, 0u, 0u, 0u});
    wave_lds_fence();
    if (member) {
        const int pos = slot_to_sample(col);   // 16 grp + r for column d_row(r, grp)
        int at[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            at[a] = cell.i[a] - win.lo[a];
            lds_put<float>(area + (first_row[a] + at[a] + grp) * kWinRow + pos * 4, grp ? cell.f[a] : kPushes ? cell.g[a] : 1.0f - cell.f[a]);
        }
        const uint8_t one = 1;
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) {
            const int a0 = axis0(pl), a1 = axis1(pl), e2 = kFlat ? 1 : win.ext[2];
            const uint32_t m = area + L::MARKS + kWinPlaneTexels * pl + ((at[a0] + grp) * win.ext[a1] + at[a1]) * e2 + (kFlat ? 0 : at[2]);
            lds_put<uint8_t>(m, one);
            lds_put<uint8_t>(m + 1, one);
            if constexpr (!kFlat) {
                lds_put<uint8_t>(m + e2, one);
                lds_put<uint8_t>(m + e2 + 1, one);
            }
        }
    }
    wave_lds_fence();

    // texels that a sample of plane pl reaches, appended to the list; scene_at: the scene's first texel in the plane's tensor
    int n_list = 0;
    auto texels_of_scene = [&](int pl) -> size_t {
        if constexpr (KIND == LP_GRID_TRIPLANE) return (size_t)g.N[axis0(pl)] * g.N[axis1(pl)];
        else if constexpr (KIND == LP_GRID_HASH) return (size_t)g.hash_size;
        else return (size_t)g.N[0] * g.N[1] * g.N[2];
    };
    auto append = [&](int pl) {
        const int a0 = axis0(pl), a1 = axis1(pl);
        const int e1 = win.ext[a1], e2 = kFlat ? 1 : win.ext[2], total = win.ext[a0] * e1 * e2;
        const float inv12 = __builtin_amdgcn_rcpf((float)(e1 * e2)), inv2 = __builtin_amdgcn_rcpf((float)e2);
        for (int n0 = 0; n0 < total; n0 += 64) {
            const int n = n0 + lane;
            const bool touched = lds_get<uint8_t>(area + L::MARKS + kWinPlaneTexels * pl + n) != 0;   // (0 behind the window)
            const unsigned long long all = __ballot(touched);
            if (touched) {
                const int t0 = small_div(n, inv12), rest = n - t0 * (e1 * e2);
                const int t1 = kFlat ? rest : small_div(rest, inv2), t2 = rest - t1 * e2;
                unsigned off;
                if constexpr (KIND == LP_GRID_TRIPLANE)
                    off = ((unsigned)(win.lo[a0] + t0) * (unsigned)g.N[a1] + (unsigned)(win.lo[a1] + t1)) * C;
                else if constexpr (KIND == LP_GRID_HASH)   // (a table whose size is a power of two; colliding texels add up)
                    off = (((unsigned)(win.lo[0] + t0) ^ (unsigned)(win.lo[1] + t1) * 2654435761u ^
                            (unsigned)(win.lo[2] + t2) * 805459861u) & (g.hash_size - 1u)) * C;
                else
                    off = (((unsigned)(win.lo[0] + t0) * (unsigned)g.N[1] + (unsigned)(win.lo[1] + t1)) * (unsigned)g.N[2] +
                           (unsigned)(win.lo[2] + t2)) * C;
                const int at = n_list + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)all, 0u));
                if constexpr (kFar)
                    lds_put<uint64_t>(area + L::WHERE + 8 * at, (uint64_t)(uintptr_t)(d_grid[pl] + scene * texels_of_scene(pl) * C) + 4ull * off);
                else
                    lds_put<uint32_t>(area + L::WHERE + 4 * at, off);
                int rows = (first_row[a0] + t0) | (first_row[a1] + t1) << 8;
                if constexpr (!kFlat) rows |= (first_row[2] + t2) << 16;
                lds_put<Which>(area + L::WHICH + L::kWhich * at, (Which)rows);
            }
            n_list += __popcll(all);
        }
    };

    // The gradient as matrix operand: lane = channel of a half (lane & 15), register k of the lanes 16 q .. 16 q + 15 =
    // position 8 q + k of the table.
    constexpr int kHalves = C / 16, kKeep = kOfRay ? 2 : 8;
    float b[kHalves][kKeep];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int k = kOfRay ? 4 * i : i;
        if constexpr (C == 32) {
            const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(dFt[k]), __float_as_uint(dFt[k + 8]), false, false);
            b[0][i] = __uint_as_float(r[0]);
            b[1][i] = __uint_as_float(r[1]);
        } else {
            float x = dFt[k], y = dFt[k + 8];
            asm("" : "+v"(x), "+v"(y));   // (or the compiler turns the choice into an indexed read of dFt)
            b[0][i] = (lane & 16) ? y : x;
        }
    }

    const int slot = lane & 15, quarter = lane >> 4;
    auto products = [&](int pl) {
        char* out = nullptr;   // the scene in plane pl's tensor
        size_t scene_at = 0;
        if constexpr (!kFar) {
            scene_at = scene * (!kFlat || pl == 0 ? texels_of_scene(0) : pl == 1 ? texels_of_scene(1) : texels_of_scene(2));
            out = reinterpret_cast<char*>((!kFlat || pl == 0 ? d_grid[0] : pl == 1 ? d_grid[1] : d_grid[2]) + scene_at * C);
        }
        [[maybe_unused]] float weight = 0.0f;
        auto rows_of = [&](int n) {   // the lane's texel (none: rows of zeros)
            return n + slot < n_list ? (int)lds_get<Which>(area + L::WHICH + L::kWhich * (n + slot)) : zero_row * 0x010101;
        };
        int rows = rows_of(0);
        for (int n0 = 0; n0 < n_list; n0 += 16) {
            const uint32_t r0 = area + (rows & 0xff) * kWinRow + 32 * quarter, r1 = area + ((rows >> 8) & 0xff) * kWinRow + 32 * quarter;
            float w[8];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const f32x4 x = lds_get<f32x4>(r0 + 16 * v), y = lds_get<f32x4>(r1 + 16 * v);
#pragma unroll
                for (int e = 0; e < 4; ++e) w[4 * v + e] = x[e] * y[e];
                if constexpr (!kFlat) {
                    const f32x4 z = lds_get<f32x4>(area + (rows >> 16) * kWinRow + 32 * quarter + 16 * v);
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[4 * v + e] *= z[e];
                }
            }
            rows = rows_of(n0 + 16);
            if constexpr (kPushes) {
                float sum = ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
                u32x2 both = __builtin_amdgcn_permlane16_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
                sum = __uint_as_float(both[0]) + __uint_as_float(both[1]);   // quarters 0 and 1, or 2 and 3
                both = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
                sum = __uint_as_float(both[0]) + __uint_as_float(both[1]);
// one add for the sums of four products, each kept by a quarter of the wave
                weight = quarter == ((n0 >> 4) & 3) ? sum : weight;
                const int n = (n0 & ~63) + lane;
                if ((n0 & 48) == 48 || n0 + 16 >= n_list)
                    if (n < n_list && weight != 0.0f) atomicAdd((!kFlat || pl == 0 ? sums[0] : pl == 1 ? sums[1] : sums[2]) + scene_at + lds_get<uint32_t>(area + L::WHERE + 4 * n) / C, weight);
            }
            if constexpr (kOfRay) {   // (a lane's eight positions are four points each of two rays)
                w[0] = (w[0] + w[1]) + (w[2] + w[3]);
                w[1] = (w[4] + w[5]) + (w[6] + w[7]);
            }
            f32x4 acc[kHalves];
#pragma unroll
            for (int h = 0; h < kHalves; ++h) acc[h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < kKeep; ++k)
#pragma unroll
                for (int h = 0; h < kHalves; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[k], b[h][k], acc[h], 0, 0, 0);
            // rows 4 quarter + p of the product (of places behind the list's end: zeros, nothing is added)
            typedef __attribute__((address_space(1))) float GlobalFloat;
            auto add = [&](GlobalFloat* at, float v) {
                if (v != 0.0f) __hip_atomic_fetch_add(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            if constexpr (kFar) {
                typedef __attribute__((__vector_size__(2 * sizeof(uint64_t)))) uint64_t u64x2;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const u64x2 o = lds_get<u64x2>(area + L::WHERE + 8 * (n0 + 4 * quarter + 2 * i));
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int h = 0; h < kHalves; ++h) add((GlobalFloat*)(uintptr_t)(o[p] + 4 * slot) + 16 * h, acc[h][2 * i + p]);
                }
            } else {
                const u32x4 o = lds_get<u32x4>(area + L::WHERE + 4 * (n0 + 4 * quarter));
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int h = 0; h < kHalves; ++h) add((GlobalFloat*)(out + 4u * (o[p] + (unsigned)slot)) + 16 * h, acc[h][p]);
            }
        }
    };

    if constexpr (kFlat) {
        // all planes at once where the list holds all their windows' texels, else one after the other
        const bool one_list = kFar && win.ext[0] * win.ext[1] + win.ext[1] * win.ext[2] + win.ext[2] * win.ext[0] <= L::kList;
        for (int from = 0; from < 3;) {
            const int to = one_list ? 3 : from + 1;
            n_list = 0;
            if (from > 0) wave_lds_fence();
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                if (pl >= from && pl < to) append(pl);
            wave_lds_fence();
            products(from);
            from = to;
        }
    } else {
        append(0);
        wave_lds_fence();
        products(0);
    }
}

// The walk on a step of the tile kernel: records and feature gradient go through LDS in the order of the
// walk (16 positions per lane group): samples of one ray in order, or ray after ray of a tile, every other
// one backwards, so that the step from ray to ray is a short one.
template <int KIND, int C, Scatter WHAT>
__device__ __forceinline__ void scatter_walk(const GridDev& g, float* const d_grid[3], float* const* sums, int scene, char* area,
                                             const Cell3& cell, bool valid, const f32x16& dFt, int lane, int full)
{
    constexpr bool kPushes = WHAT != Scatter::kGradient, kOfRay = WHAT == Scatter::kPushRay;
    const int col = lane & 31, grp = lane >> 5;
    auto flip = [full](int c) { return (c & full) ? c ^ (full - 1) : c; };   // column <-> position of the walk
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
// `full`: samples of a ray in the step.  Steps of a single ray: see RayWindows; `windows` false: the walk.
template <int KIND, int C, Scatter WHAT = Scatter::kGradient, RayWindows RAYS = WHAT == Scatter::kGradient ? RayWindows::kSplit : RayWindows::kNone>
__device__ __forceinline__ void scatter_step(const GridDev& g, float* const d_grid[3], int scene, uint32_t area,
                                             char* area_ptr, const Cell3& cell, const f32x16& dFt, int lane, int full,
                                             float* const* sums = nullptr, bool valid = true, bool windows = true)
{
    constexpr bool kOfRay = WHAT == Scatter::kPushRay;
    const int k = lane & (full - 1);
    const bool tile = full < 32;
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
        scatter_walk<KIND, C, WHAT>(g, d_grid, sums, scene, area_ptr, cell, valid, dFt, lane, full);
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

// Whether the rays that the lanes name run side by side: in one scene, and within APART cells of the first lane's at both ends.
template <int APART = 3, class CellOf>
__device__ __forceinline__ bool side_by_side(const RaysDev& rays, long long ray, CellOf cell_of)
{
    const RayGeom q = load_ray_geom(rays, ray);
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
