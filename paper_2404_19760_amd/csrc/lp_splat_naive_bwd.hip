// Naive Splatter backward (Section 3.3 "Splatter"): the gradient of a pixel's feature is the normalised
// output gradient read at every point of its ray and summed,
//     d_feats[ray] = sum over points and corners of weight / theta_w[corner] * d_theta[corner].
//
// What bounds it: the texel reads (the caches return 64 bytes a cycle and compute unit). Nothing has to be known
// per point, so the lanes of a wave are the 16-byte pieces of texels: 64 points publish a normalised weight and a byte
// offset per corner in LDS, then each load instruction reads 8 (16 channels: 16) whole texels, every lane keeps the
// sum of what it read over the whole ray, and the corners meet once per ray.
// Large images are taken in patches of 4 x 4 pixels (lp_splat_patch.h): a texel is read once for the step's 128 points, 0.75
// reads per point instead of eight, and a matrix product hands it to the rays; then instructions bound it (two waves a SIMD).
// 160^3 x 32 voxels, 4 x 128^2 rays x 160 points: 5.86 ms with a lane per ray (lp_generic.hip), 0.51 ms by texel pieces, 0.44 ms
// in patches (0.38 with sums in fp32, further from 64 bits than ray by ray: pull_points; in patches of 8 x 4 pixels, whose weights
// leave room for one wave a SIMD, twice as long).
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_splat_common.h"
#include "lp_splat_patch.h"
#include "lp_tile_lds.h"

namespace lp {

namespace {

constexpr int kWaves = 4;
constexpr int kPoints = 64;      // points whose records stand in LDS at a time
constexpr int kPatchRays = 16;   // of a patch: see lp_splat_patch.h
using Patch = PatchLds<kPatchRays>;
constexpr int kPointUnit = 32;   // they are read in multiples of this many (the rest: weight zero)

typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(2 * sizeof(double)))) double f64x2;

template <int KIND>
struct PushRecords {
    static constexpr int kPlanes = KIND == LP_GRID_TRIPLANE ? 3 : 1;
    static constexpr int kCorners = KIND == LP_GRID_TRIPLANE ? 4 : 8;   // of a plane's cell
    static constexpr int kPoint = kCorners * 8;                         // bytes: (weight, byte offset) per corner
    static constexpr int kPlane = kPoints * kPoint;
    static constexpr int kBytes = kPlanes * kPlane;
};

// LDS of a patch's wave: two arrays of a float per slot take the map's place and a little more, then the rays' sums, up to eight to a lane
constexpr int kTotals = Patch::MAP + Patch::kSlots * 8;
constexpr int kPatchBytes = kTotals + 64 * 8 * 8;
static_assert(kTotals >= Patch::kBytes && kTotals % 16 == 0, "the map");
static_assert(2 * kWaves * kPatchBytes <= 160 * 1024, "the LDS of two workgroups fits a compute unit");

// Weights over the weight sums of the forward (0 where nothing landed, and past the ray's end) and texel
// offsets of the lane's point.
template <int KIND, int C>
__device__ __forceinline__ void publish_normalised(uint32_t at, const GridDev& tgt, const SplatDev& sp, int scene,
                                                   const Cell3& c, bool valid)
{
    using Rec = PushRecords<KIND>;
#pragma unroll
    for (int p = 0; p < Rec::kPlanes; ++p) {
        float w[Rec::kCorners];
        unsigned cell[Rec::kCorners];
        const float* W;
        if constexpr (KIND == LP_GRID_TRIPLANE) {
            const int a = p, b = (p + 1) % 3;
            W = sp.theta_w_in[p] + (size_t)scene * tgt.N[a] * tgt.N[b];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int da = d >> 1, db = d & 1;
                w[d] = (da ? c.f[a] : c.g[a]) * (db ? c.f[b] : c.g[b]);
                cell[d] = (unsigned)(c.i[a] + da) * (unsigned)tgt.N[b] + (unsigned)(c.i[b] + db);
            }
        } else {
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const int dx = d >> 2, dy = (d >> 1) & 1, dz = d & 1;
                w[d] = (dx ? c.f[0] : c.g[0]) * (dy ? c.f[1] : c.g[1]) * (dz ? c.f[2] : c.g[2]);
                if constexpr (KIND == LP_GRID_VOXEL)
                    cell[d] = ((unsigned)(c.i[0] + dx) * (unsigned)tgt.N[1] + (unsigned)(c.i[1] + dy)) * (unsigned)tgt.N[2] +
                              (unsigned)(c.i[2] + dz);
            }
            if constexpr (KIND == LP_GRID_HASH) {
                hash_corner_slots(c, tgt.hash_size, cell);
                W = sp.theta_w_in[0] + (size_t)scene * tgt.hash_size;
            } else {
                W = sp.theta_w_in[0] + (size_t)scene * tgt.N[0] * tgt.N[1] * tgt.N[2];
            }
        }
        float ws[Rec::kCorners];
#pragma unroll
        for (int d = 0; d < Rec::kCorners; ++d) ws[d] = W[cell[d]];
#pragma unroll
        for (int d = 0; d < Rec::kCorners; d += 2) {
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                v[2 * e] = __float_as_uint((valid && ws[d + e] > 0.0f) ? w[d + e] / ws[d + e] : 0.0f);
                v[2 * e + 1] = cell[d + e] * (C * 4u);
            }
            lds_put<u32x4>(at + p * Rec::kPlane + 8 * d, v);
        }
    }
}

// One ray; `area`: PushRecords<KIND>::kBytes of LDS of the wave.
template <int KIND, int C, bool CC>
__device__ __forceinline__ void ray_gradient(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, long long ray, uint32_t area,
                                             int lane)
{
    using Rec = PushRecords<KIND>;
    constexpr int kLanes = C / 4;            // lanes of a texel
    constexpr int kTexels = 64 / kLanes;     // texels of a load
    constexpr int kUnroll = 8;
    static_assert(kPointUnit * Rec::kCorners % (kTexels * kUnroll) == 0, "whole unrolled rounds");
    const uint32_t mine = area + (lane / kLanes) * 8;
    const uint32_t piece = (lane % kLanes) * 16;
    const int S = rays.S;
    const RayGeom q = load_ray_geom(rays, ray);
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int j0 = 0; j0 < S; j0 += kPoints) {
        const int j = j0 + lane;
        const Cell3 c = sample_cell<CC>(tgt, q, min(j, S - 1));
        wave_lds_fence();
        publish_normalised<KIND, C>(area + lane * Rec::kPoint, tgt, sp, q.scene, c, j < S);
        wave_lds_fence();
        const int points = min((S - j0 + kPointUnit - 1) / kPointUnit * kPointUnit, kPoints);
#pragma unroll
        for (int p = 0; p < Rec::kPlanes; ++p) {
            const char* G = reinterpret_cast<const char*>(sp.d_theta[p] + scene_texel<KIND>(tgt, p, q.scene) * C);
            const int end = points * Rec::kPoint, live = (S - j0) * Rec::kPoint;
            for (int at = 0; at < end; at += kUnroll * kTexels * 8) {
                u32x2 rec[kUnroll];
                f32x4 x[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) rec[u] = lds_get<u32x2>(mine + p * Rec::kPlane + at + u * kTexels * 8);
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) x[u] = *reinterpret_cast<const f32x4*>(G + (rec[u][1] + piece));
                if (at + kUnroll * kTexels * 8 > live) {   // past the ray's end: nothing, also where the texel is infinite
#pragma unroll
                    for (int u = 0; u < kUnroll; ++u)
                        if (at + (u * kTexels + lane / kLanes) * 8 >= live) x[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] += __uint_as_float(rec[u][0]) * x[u][e];
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int d = kLanes; d < 64; d <<= 1) sum[e] += __shfl_xor(sum[e], d, 64);
    if (lane < kLanes) {
        const f32x4 v = {sum[0], sum[1], sum[2], sum[3]};
        *reinterpret_cast<f32x4*>(sp.d_feats + (size_t)ray * C + 4 * lane) = v;
    }
}

// Patches are taken from this many rays on, where points share texels: up to `longest` texels from point to point.  Time ray by ray over
// that in patches, 62^3 .. 233^3 voxels, 64 to 130 points a ray: 1.09 .. 1.6 at 160 000 rays (ten thousand patches for two thousand
// waves); at 65 536 and 90 000 rays with 16 channels 1.00 .. 1.28 up to 0.75 texels and 0.83 .. 1.02 beyond, with 32 channels 1.10 ..
// 1.7 up to 1.25 and 0.88 .. 1.09 beyond; 0.7 .. 1.3 at 16 384.  Looking for an image takes 7 us, 8 % of 1.6e6 points ray by ray.
// Triplanes stay ray by ray (0.3 .. 1.4).  And from this many points times channels on: with fewer the sums of a ray in its lanes,
// S C / 32 terms long each, are nearer to 64 bits (2-norm of the error at 24 points: 16 channels 0.90e-7, in patches 0.97e-7; 32
// channels 0.96e-7 and 0.94e-7).
constexpr long long kMinRays = 65536, kMinPoints = 4000000, kManyRays = 131072;
constexpr int kMinPointChannels = 768;
template <int C>
__device__ __forceinline__ long long image_row(const GridDev& g, const RaysDev& rays)
{
    const double longest = rays.M >= kManyRays ? 2.0 : C == 16 ? 0.75 : 1.25;
    __shared__ int found;
    return find_row(g, rays, 0.9, longest, found);
}

// Rays in their order.  PATCHES: the patch kernel has been launched before and takes what it finds to be an image.
template <int KIND, int C, bool CC, bool PATCHES>
__global__ __launch_bounds__(kWaves * 64) void splat_naive_bwd_kernel(GridDev tgt, RaysDev rays, SplatDev sp)
{
    __shared__ __align__(16) char records[kWaves][PushRecords<KIND>::kBytes];
    if constexpr (PATCHES) {
        if (image_row<C>(tgt, rays) != 0) return;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)records[wave];
    const RaySchedule sched = ray_schedule(rays.M, kWaves);
    for (long long ray = sched.first; ray < sched.end; ray += sched.stride) ray_gradient<KIND, C, CC>(tgt, rays, sp, ray, area, lane);
}

// Where a lane keeps the sums of its registers r and r + 1 of channel block h.
__device__ __forceinline__ uint32_t total_at(uint32_t area, int h, int r, int lane)
{
    uint32_t lane_here = lane;   // (an address kept beside the texels of a step would cost spills)
    refresh(lane_here);
    return area + kTotals + 1024 * (2 * h + r / 2) + 16 * lane_here;
}

// The gradient of a patch's pixels, d_feat[ray][channel] += weights[texel][ray] / theta_w[texel] x d_theta[texel][channel],
// for points [from, from + len) of a step, plane `pl` (`only`: of one ray).  false: they reach too many texels.
// A product takes four texels; lane quarter q of a round of 32 texels reads texels 8 q .. 8 q + 7, two neighbouring channels of
// each (16 channels: one).  `probe` becomes undefined where a gradient that was read is not finite.
// Products in fp32, in two chains to a round, and the sums of the rounds in fp64: one fp32 chain through all texels of a ray, with
// weights times reciprocals, was two to three times as far from 64 bits as the sums that the lanes keep ray by ray (2-norm at 160
// points, 32 channels: 2.9e-7 against 1.3e-7; this way 0.8e-7, for 13 % of the time).
template <int KIND, int C>
__device__ __forceinline__ bool pull_points(const GridDev& g, const SplatDev& sp, int scene, uint32_t area, const PatchCells& cells,
                                            int from, int len, int only, int pl, float& probe, int lane)
{
    constexpr int kRounds = Patch::kSlots / 32, kVec = C / 16;
    const int n_slots = patch_weights<KIND, C, kPatchRays>(area, g, cells, from, len, only, pl, lane);
    if (n_slots <= 0) return n_slots == 0;
    const size_t scene_at = scene_texel<KIND>(g, pl, scene);
    const float* W = sp.theta_w_in[pl] + scene_at;
    const int i16 = lane & 15, q = lane >> 4;
    const char* G = reinterpret_cast<const char*>(sp.d_theta[pl] + scene_at * C) + 4 * kVec * i16;
    // up to a whole round: the last texel again, with weight zero
    if (lane < 32 && n_slots + lane < Patch::kSlots)
        lds_put<uint32_t>(area + Patch::OFFSETS + 4 * (n_slots + lane), lds_get<uint32_t>(area + Patch::OFFSETS + 4 * (n_slots - 1)));
    wave_lds_fence();
    // all of the step's reads are under way before the first is waited for; the weight sums first
    float sums[(Patch::kSlots + 63) / 64];
#pragma unroll
    for (int n = 0; n < (Patch::kSlots + 63) / 64; ++n) {
        if (64 * n >= n_slots) break;
        sums[n] = W[lds_get<uint32_t>(area + Patch::OFFSETS + 4 * min(64 * n + lane, n_slots - 1)) / C];
    }
    float x[kRounds][8][kVec];
#pragma unroll
    for (int n = 0; n < kRounds; ++n) {
        if (32 * n >= n_slots) break;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const u32x4 off = lds_get<u32x4>(area + Patch::OFFSETS + 4 * (32 * n + 8 * q + 4 * v));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float* at = reinterpret_cast<const float*>(G + 4u * off[e]);
                if constexpr (kVec == 2) {
                    const f32x2 y = *reinterpret_cast<const f32x2*>(at);
                    x[n][4 * v + e][0] = y[0];
                    x[n][4 * v + e][kVec - 1] = y[1];
                } else {
                    x[n][4 * v + e][0] = *at;
                }
            }
        }
    }
    // theta_w and 1 / theta_w (0 where nothing landed).  Tiny sums are multiplied by a power of two that keeps the reciprocal
    // finite, and stand there with a minus sign.
    constexpr int SUM = Patch::MAP, INVERSE = Patch::MAP + Patch::kSlots * 4;
    constexpr float kTiny = 0x1p-100f, kScale = 0x1p80f;
#pragma unroll
    for (int n = 0; n < (Patch::kSlots + 63) / 64; ++n) {
        if (64 * n >= n_slots) break;
        if (64 * n + lane < Patch::kSlots) {
            const float w = sums[n], scaled = w < kTiny ? w * kScale : w;
            const bool there = 64 * n + lane < n_slots && w > 0.0f;
            lds_put<float>(area + SUM + 4 * (64 * n + lane), w < kTiny ? -scaled : scaled);
            lds_put<float>(area + INVERSE + 4 * (64 * n + lane), there ? 1.0f / scaled : 0.0f);
        }
    }
    wave_lds_fence();
#pragma unroll
    for (int n = 0; n < kRounds; ++n) {
        if (32 * n >= n_slots) break;
        f32x4 part_sum[2][C / 16];
#pragma unroll
        for (int h = 0; h < C / 16; ++h) { part_sum[0][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; part_sum[1][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int mine = 32 * n + 8 * q + 4 * v;
            const f32x4 sum = lds_get<f32x4>(area + SUM + 4 * mine), inverse = lds_get<f32x4>(area + INVERSE + 4 * mine);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float part = lds_get<float>(area + min(mine + e, n_slots - 1) * Patch::kRow + 4 * i16) * (sum[e] < 0.0f ? kScale : 1.0f);
                const float about = part * inverse[e], w = fmaf(fmaf(-about, fabsf(sum[e]), part), inverse[e], about);   // part / sum, rounded once
#pragma unroll
                for (int h = 0; h < kVec; ++h) {
                    probe = fmaf(x[n][4 * v + e][h], 0.0f, probe);
                    part_sum[e & 1][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, x[n][4 * v + e][h], part_sum[e & 1][h], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int h = 0; h < C / 16; ++h)
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                const uint32_t at = total_at(area, h, r, lane);
                f64x2 t = lds_get<f64x2>(at);
#pragma unroll
                for (int i = 0; i < 2; ++i) t[i] += (double)part_sum[0][h][r + i] + (double)part_sum[1][h][r + i];
                lds_put<f64x2>(at, t);
            }
    }
    return true;
}

// Images, patch after patch (lp_splat_patch.h).  A part of a patch whose rays are not neighbours or not finite, or that reads a
// gradient that is not (a product would spread it over all of its rays), is taken ray by ray.
template <int KIND, int C, bool CC>
__global__ __launch_bounds__(kWaves * 64, 2) void splat_patch_bwd_kernel(GridDev tgt, RaysDev rays, SplatDev sp)
{
    extern __shared__ uint4 lds_raw[];
    const long long row = image_row<C>(tgt, rays);
    if (row == 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)(reinterpret_cast<char*>(lds_raw) + wave * kPatchBytes);
    static_assert(PushRecords<KIND>::kBytes <= kPatchBytes, "the records of a ray");   // (taken ray by ray a part has no sums)
    constexpr int kPlanes = PushRecords<KIND>::kPlanes;
    const PatchGrid<kPatchRays> grid(rays.M, row);
    const int S = rays.S;
    const RaySchedule sched = ray_schedule(grid.count, kWaves);
    for (long long patch = sched.first; patch < sched.end; patch += sched.stride) {
        constexpr int kW = PatchGrid<kPatchRays>::kW;
        auto my_ray = [&](bool& there) {
            uint32_t lane_here = lane;   // (loaded for every part anew: kept beside the texels of a step it would cost spills)
            refresh(lane_here);
            return load_ray_geom(rays, grid.ray(patch, lane_here & (kPatchRays - 1), there));
        };
        unsigned lines;
        {
            bool there;
            const RayGeom q = my_ray(there);
            lines = patch_lines<kPatchRays, CC>(tgt, q, there, S, lane);
        }
        patch_parts(lines, [&](int y0, int y1, bool by_rays) {
            bool there;
            const RayGeom q = my_ray(there);
            const int y = (lane & (kPatchRays - 1)) / kW;
            const bool ok = there && y >= y0 && y < y1;
            const unsigned long long oks = __ballot(ok);
            if (oks == 0ull) return;
            bool whole = !by_rays;
#pragma unroll
            for (int h = 0; h < C / 16; ++h)
#pragma unroll
                for (int r = 0; r < 4; r += 2) lds_put<f64x2>(total_at(area, h, r, lane), f64x2{0.0, 0.0});
            if (whole) {
                const int scene = __builtin_amdgcn_readfirstlane(__shfl(q.scene, __builtin_ctzll(oks), 64));
                float probe = 0.0f;
                for (int j0 = 0; j0 < S; j0 += kPatchPoints) {
                    const PatchCells cells = patch_cells<CC>(tgt, q, ok, j0, S, S);
#pragma unroll 1
                    for (int pl = 0; pl < kPlanes; ++pl)
                        patch_steps<kPatchRays>([&](int from, int len, int only) {
                            return pull_points<KIND, C>(tgt, sp, scene, area, cells, from, len, only, pl, probe, lane);
                        });
                }
                whole = __ballot(probe != 0.0f) == 0ull;
            }
            for (int i = kW * y0; i < kW * y1; ++i) {
                if (whole) break;
                bool has;
                const long long at = grid.ray(patch, i, has);
                if (has) ray_gradient<KIND, C, CC>(tgt, rays, sp, at, area, lane);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {   // register r: ray 4 (lane / 16) + r, the lane's channels
                bool has;
                const long long at = grid.ray(patch, 4 * (lane >> 4) + r, has);
                if (!whole || !has || (lane >> 4) < y0 || (lane >> 4) >= y1) continue;
                float* out = sp.d_feats + (size_t)at * C + C / 16 * (lane & 15);
                auto sum = [&](int h) { return (float)lds_get<f64x2>(total_at(area, h, r & 2, lane))[r & 1]; };
                if constexpr (C == 32) *reinterpret_cast<f32x2*>(out) = f32x2{sum(0), sum(1)};
                else *out = sum(0);
            }
            wave_lds_fence();
        });
    }
}

template <int KIND, int C, bool CC>
hipError_t launch_t(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    constexpr bool kMayPatch = KIND != LP_GRID_TRIPLANE;
    const bool patches = kMayPatch && rays.M >= kMinRays && rays.M * rays.S >= kMinPoints && rays.S * C >= kMinPointChannels;
    if constexpr (kMayPatch) if (patches) {
        auto kernel = splat_patch_bwd_kernel<KIND, C, CC>;
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kWaves * kPatchBytes);
        if (e != hipSuccess) return e;
        const long long blocks = (2LL * n_cu + 7) / 8 * 8;   // the LDS of two workgroups fits a compute unit
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kWaves * 64), kWaves * kPatchBytes, stream, tgt, rays, sp);
    }
    long long blocks = 6LL * n_cu;   // the LDS of six workgroups fits a compute unit for every structure
    const long long need = (rays.M + kWaves - 1) / kWaves;
    if (blocks > need) blocks = need;
    blocks = (blocks + 7) / 8 * 8;
    auto kernel = patches ? splat_naive_bwd_kernel<KIND, C, CC, kMayPatch> : splat_naive_bwd_kernel<KIND, C, CC, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kWaves * 64), 0, stream, tgt, rays, sp);
    return hipGetLastError();
}

template <int KIND, int C>
hipError_t launch(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    return tgt.contract > 0.0 ? launch_t<KIND, C, true>(tgt, rays, sp, n_cu, stream) : launch_t<KIND, C, false>(tgt, rays, sp, n_cu, stream);
}

template <int KIND>
hipError_t dispatch(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    return tgt.C == 16 ? launch<KIND, 16>(tgt, rays, sp, n_cu, stream) : launch<KIND, 32>(tgt, rays, sp, n_cu, stream);
}

}  // namespace

bool splat_naive_bwd_supported(const GridDev& tgt, const SplatDev& sp)
{
    if (!splat_naive_supported(tgt)) return false;
    for (int p = 0; p < (tgt.kind == LP_GRID_TRIPLANE ? 3 : 1); ++p)
        if ((uintptr_t)sp.d_theta[p] & 15u) return false;   // 16-byte loads
    return ((uintptr_t)sp.d_feats & 15u) == 0;
}

hipError_t launch_splat_naive_bwd(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu,
                                  hipStream_t stream)
{
    if (tgt.kind == LP_GRID_HASH) return dispatch<LP_GRID_HASH>(tgt, rays, sp, n_cu, stream);
    return tgt.kind == LP_GRID_VOXEL ? dispatch<LP_GRID_VOXEL>(tgt, rays, sp, n_cu, stream)
                                     : dispatch<LP_GRID_TRIPLANE>(tgt, rays, sp, n_cu, stream);
}

}  // namespace lp
