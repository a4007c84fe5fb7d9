// Naive Splatter backward (Section 3.3 "Splatter"): the gradient of a pixel's feature is the normalised
// output gradient read at every point of its ray and summed,
//     d_feats[ray] = sum over points and corners of weight / theta_w[corner] * d_theta[corner].
//
// What bounds it: the texel reads (the caches return 64 bytes a cycle and compute unit). Nothing has to be known
// per point, so the lanes of a wave are the 16-byte pieces of texels: 64 points publish a normalised weight and a byte
// offset per corner in LDS, then each load instruction reads 8 (16 channels: 16) whole texels, every lane keeps the
// sum of what it read over the whole ray, and the corners meet once per ray.
// 160^3 x 32 voxels, 4 x 128^2 rays x 160 points: 5.86 ms with a lane per ray (lp_generic.hip) -> 0.52 ms.
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_splat_common.h"
#include "lp_tile_lds.h"

namespace lp {

namespace {

constexpr int kWaves = 4;
constexpr int kPoints = 64;      // points whose records stand in LDS at a time
constexpr int kPointUnit = 32;   // they are read in multiples of this many (the rest: weight zero)

template <int KIND>
struct PushRecords {
    static constexpr int kPlanes = KIND == LP_GRID_TRIPLANE ? 3 : 1;
    static constexpr int kCorners = KIND == LP_GRID_TRIPLANE ? 4 : 8;   // of a plane's cell
    static constexpr int kPoint = kCorners * 8;                         // bytes: (weight, byte offset) per corner
    static constexpr int kPlane = kPoints * kPoint;
    static constexpr int kBytes = kPlanes * kPlane;
};

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

template <int KIND, int C, bool CC>
__global__ __launch_bounds__(kWaves * 64) void splat_naive_bwd_kernel(GridDev tgt, RaysDev rays, SplatDev sp)
{
    using Rec = PushRecords<KIND>;
    constexpr int kLanes = C / 4;            // lanes of a texel
    constexpr int kTexels = 64 / kLanes;     // texels of a load
    constexpr int kUnroll = 8;
    static_assert(kPointUnit * Rec::kCorners % (kTexels * kUnroll) == 0, "whole unrolled rounds");
    __shared__ __align__(16) char records[kWaves][Rec::kBytes];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)records[wave];
    const uint32_t mine = area + (lane / kLanes) * 8;
    const uint32_t piece = (lane % kLanes) * 16;

    const RaySchedule sched = ray_schedule(rays.M, kWaves);
    const int S = rays.S;
    for (long long ray = sched.first; ray < sched.end; ray += sched.stride) {
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
                const char* G;
                if constexpr (KIND == LP_GRID_TRIPLANE)
                    G = reinterpret_cast<const char*>(sp.d_theta[p] + (size_t)q.scene * tgt.N[p] * tgt.N[(p + 1) % 3] * C);
                else if constexpr (KIND == LP_GRID_HASH)
                    G = reinterpret_cast<const char*>(sp.d_theta[0] + (size_t)q.scene * tgt.hash_size * C);
                else
                    G = reinterpret_cast<const char*>(sp.d_theta[0] + (size_t)q.scene * tgt.N[0] * tgt.N[1] * tgt.N[2] * C);
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
}

template <int KIND, int C>
hipError_t launch(const GridDev& tgt, const RaysDev& rays, const SplatDev& sp, int n_cu, hipStream_t stream)
{
    long long blocks = 6LL * n_cu;   // the LDS of six workgroups fits a compute unit for every structure
    const long long need = (rays.M + kWaves - 1) / kWaves;
    if (blocks > need) blocks = need;
    blocks = (blocks + 7) / 8 * 8;
    if (tgt.contract > 0.0)
        hipLaunchKernelGGL((splat_naive_bwd_kernel<KIND, C, true>), dim3((unsigned)blocks), dim3(kWaves * 64), 0, stream, tgt, rays, sp);
    else
        hipLaunchKernelGGL((splat_naive_bwd_kernel<KIND, C, false>), dim3((unsigned)blocks), dim3(kWaves * 64), 0, stream, tgt, rays, sp);
    return hipGetLastError();
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
