// Matrix-core forward kernel of the Renderer (Eq. (1), Section 3.3; fused as in Section 3.4).
//
// A workgroup is 4 wavefronts sharing the MLP weights in LDS (bf16 hi/lo MFMA A operands).
// A wavefront marches two neighbouring rays, 32 consecutive samples of each per step, or one ray, 64 samples per step; sampled by
// whole texels (lp_gather.h) or with lanes (i, g) interpolating the g-th half of the channels of samples i of both halves of the
// step; the MLP runs on the
// matrix cores for the 64 samples (two N blocks of 32, a stage apart), then lane l owns sample l of the step
// for the density / colour heads and the emission-absorption update, where the transmittance
// prefix is a scan of sigma * Delta over the lanes of a ray.  Nothing per sample is written to memory.
// What bounds it: instruction issue (256^3 x 16 voxels in bf16, 563 563 rays x 330 samples: 984 wave instructions on the vector ALU
// a step, the products among them, issue in 80 % of a SIMD's cycles and the matrix cores are busy in 49 %).  So rays come in pairs,
// which leaves fewer places empty at their ends (330 samples: 6 % instead of 14 %), each lane forms the cell of one sample and the
// halves of the wave exchange them, and a load's address is a uniform pointer and the lane's offset: 9.57 -> 8.46 ms.  And more
// workgroups than fit at once (launch_items): 8.52 -> 7.54.
#include "lp_gather.h"
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"

#include <algorithm>
#include <type_traits>

namespace lp {

namespace {

constexpr int kWaves = 4;

// Whether the wave samples by whole texels (lp_gather.h): 32 grid channels, any structure but a HexPlane (measured: eight
// 256^2 triplanes 46.3 -> 28.6 ms, 64^3 voxels 3.0 -> 2.4, 160^3 with contract coordinates 1.98 -> 1.52). With 16
// channels the texels take a quarter or a third of those loads and the kernel is bound by the MLP: a lane per
// sample is then the cheaper one (256^3 voxels 14.05 against 14.2 ms, stored in bf16 9.45 against 9.57).
template <int KIND, int C, int CG>
constexpr bool kWaveGather = C == 32 && CG == C && KIND != LP_GRID_HEXPLANE;

// LDS: the MLP, then (16-byte units from kGatherAt) the waves' gather areas, then (PAIRS) their rays.
template <int KIND, int C, int H, int NH, int CG, bool PAIRS>
struct FwdLds {
    static constexpr int kGatherAt = (MlpLds<C, H, NH, false, 2>::END + 15) / 16 * 16;
    static constexpr int kWave = kWaveGather<KIND, C, CG> ? WaveGatherLds<KIND == LP_GRID_HEXPLANE ? LP_GRID_VOXEL : KIND, CG>::kBytes : 0;
    static constexpr int kRays = PAIRS ? 2 * 48 : 0;   // of a wave: the geometry of its two rays
    static constexpr int RAYS_AT = kGatherAt * 16 + kWaves * kWave;
    static constexpr int kBytes = RAYS_AT + kWaves * kRays;
    static_assert(RAYS_AT % 16 == 0, "alignment");
};

// Whether the kernel can take rays in pairs (the direction inputs of two rays and a HexPlane's reads leave no registers).
template <int KIND, int C, int CG>
constexpr bool kPairs = CG == C && KIND != LP_GRID_HEXPLANE;

// Lane l owns sample l of a step: of 64 samples of a ray, or (PAIRS) of 32 of ray l / 32 of two.
// (three waves per SIMD where the registers allow it without spilling)
template <int KIND, int C, int H, int NH, bool CC, int CG, int GT, bool PAIRS>
__global__ __launch_bounds__(kWaves * 64, (kPairs<KIND, C, CG> ? 3 : 1)) void fwd_mfma_kernel(GridDev g, MlpDev m, RaysDev rays, FwdOut out)
{
    static_assert(!PAIRS || kPairs<KIND, C, CG>);
    constexpr int kLanes = PAIRS ? 32 : 64;   // of a ray: its samples of a step
    using L = MlpLds<C, H, NH, false, 2>;
    using F = FwdLds<KIND, C, H, NH, CG, PAIRS>;
    extern __shared__ uint4 lds[];
    stage_mlp<C, H, NH, false, 2, CG>(lds, m);
    __syncthreads();

    const int lane = threadIdx.x & 63, half = PAIRS ? lane >> 5 : 0;
    const RaySchedule sched = ray_schedule(PAIRS ? (rays.M + 1) / 2 : rays.M, kWaves);
    const int S = rays.S;
    const bool identity = m.feat_act != 0;   // rendered features without the sigmoid (two-MLP decoder only)
    const uint32_t area = (uint32_t)(uintptr_t)(LdsByte*)reinterpret_cast<char*>(lds) + F::kGatherAt * 16 +
                          __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * F::kWave;
    const uint32_t ray_at = (uint32_t)(uintptr_t)(LdsByte*)reinterpret_cast<char*>(lds) + F::RAYS_AT + (threadIdx.x >> 5) * (F::kRays / 2);

    for (long long item = sched.first; item < sched.end; item += sched.stride) {
        const long long ray = PAIRS ? 2 * item : item;   // the first one
        RayGeom q0 = load_ray_geom(rays, ray);
        if constexpr (CG != C) set_direction_inputs(m, q0);
        const RayGeom q1 = PAIRS ? load_ray_geom(rays, min(ray + 1, rays.M - 1)) : q0;
        if constexpr (PAIRS) {
            wave_lds_fence();
            if ((lane & 31) == 0) {   // each half's ray
                const RayGeom& q = half ? q1 : q0;
                lds_put<f32x4>(ray_at, f32x4{q.ox, q.oy, q.oz, q.dx});
                lds_put<f32x4>(ray_at + 16, f32x4{q.dy, q.dz, q.near, q.delta});
                lds_put<double>(ray_at + 32, q.delta64);
            }
            wave_lds_fence();
        }
        // optical depth of earlier steps; in pairs, which have twice as many of them, summed in fp64
        typename std::conditional<PAIRS, double, float>::type tau = 0;
        float acc_r = 0.0f, acc_g = 0.0f, acc_b = 0.0f, acc_d = 0.0f;  // per-lane partial sums

        for (int j0 = 0; j0 < S; j0 += kLanes) {
            const int j = j0 + (lane & (kLanes - 1));
            struct { float z[4]; } a;
            // the samples' cells, column lane % 32 of both N blocks
            Cell3 pair[2];
            if constexpr (PAIRS) {
                RayGeom q;   // the lane's ray (from LDS: kept in registers it would cost ten, or twenty converted to fp64 ahead of the loop)
                uint32_t at = ray_at;
                refresh(at);
                const f32x4 u = lds_get<f32x4>(at), v = lds_get<f32x4>(at + 16);
                q.ox = u[0]; q.oy = u[1]; q.oz = u[2]; q.dx = u[3]; q.dy = v[0]; q.dz = v[1]; q.near = v[2]; q.delta = v[3];
                q.delta64 = lds_get<double>(at + 32);
                block_cells(sample_cell_for<CC, GT>(g, q, min(j, S - 1)), pair);
            }
            auto cell = [&](int nb) {
                if constexpr (PAIRS) return pair[nb];
                else return sample_cell_for<CC, GT>(g, q0, min(j0 + 32 * nb + (lane & 31), S - 1));
            };
            if constexpr (kWaveGather<KIND, C, CG>) {
                using G = WaveGatherLds<KIND, C>;
                Frag fh[2][C / 16], fl[2][C / 16];
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    wave_features<KIND, C, GT>(g, nb ? q1.scene : q0.scene, cell(nb), area, area + G::IMG, lane, fh[nb], fl[nb]);
                mlp_outputs<C, H, NH>(lds, reinterpret_cast<const float*>(lds + L::BIAS), lane, fh, fl, a.z);
            } else {
                forward_outputs<KIND, C, H, NH, CG, GT>(g, lds, q0, q1, cell, lane, a.z);
            }

            // heads and emission-absorption update
            float near = q0.near, delta = q0.delta;
            if constexpr (PAIRS) {
                uint32_t at = ray_at;
                refresh(at);
                near = lds_get<float>(at + 24);
                delta = lds_get<float>(at + 28);
            }
            const float t = near + ((float)j + 0.5f) * delta;
            const float sd = j < S ? fast_softplus(a.z[0]) * delta : 0.0f;
            const float incl = group_scan_incl<kLanes>(sd, lane);
            const float Tprev = __expf(-(float)(tau + (incl - sd)));
            const float w = Tprev * one_minus_exp_neg(sd);
            acc_r += w * feature_head(a.z[1], identity);
            acc_g += w * feature_head(a.z[2], identity);
            acc_b += w * feature_head(a.z[3], identity);
            acc_d += w * t;
            tau += __shfl(incl, kLanes - 1, kLanes);
        }

        auto ray_sum = [&](float v) {
#pragma unroll
            for (int k = kLanes / 2; k > 0; k >>= 1) v += __shfl_xor(v, k, 64);
            return v;
        };
        acc_r = ray_sum(acc_r);
        acc_g = ray_sum(acc_g);
        acc_b = ray_sum(acc_b);
        acc_d = ray_sum(acc_d);
        if (lane == 0 || (PAIRS && lane == 32 && ray + 1 < rays.M)) {
            const long long r = ray + half;
            const float depth = (float)tau, T = __expf(-depth);
            out.rgb[3 * r + 0] = acc_r + T * out.bg[0];
            out.rgb[3 * r + 1] = acc_g + T * out.bg[1];
            out.rgb[3 * r + 2] = acc_b + T * out.bg[2];
            if (out.alpha) out.alpha[r] = one_minus_exp_neg(depth);
            if (out.depth) out.depth[r] = acc_d;
            if (out.cache) out.cache[r] = depth;
        }
    }
}

template <int KIND, int C, int H, int NH, bool CC, int CG, int GT, bool PAIRS>
hipError_t launch_items(const GridDev& g, const MlpDev& m, const RaysDev& rays, const FwdOut& out, long long blocks, hipStream_t stream)
{
    constexpr int kLdsBytes = FwdLds<KIND, C, H, NH, CG, PAIRS>::kBytes;
    auto kernel = fwd_mfma_kernel<KIND, C, H, NH, CC, CG, GT, PAIRS>;
    const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
    const long long items = PAIRS ? (rays.M + 1) / 2 : rays.M, need = (items + kWaves - 1) / kWaves;
    // More workgroups than fit at once, where each still has work for longer than its staging takes: a SIMD serves its oldest wave first, so
    // that of three workgroups of equal work the first was done early and the last ran alone; now others follow. 32 steps to a wave: 563 563 rays x
    // 330 samples, 256^3 x 16 voxels in bf16, 8.62 -> 7.88 ms (16 steps 7.99, 64 steps 7.97), 64^3 x 32 voxels 2.43 -> 2.33,
    // eight triplanes 26.2 -> 25.5; one step or two to a wave (5003 rays x 193 samples) took 6 % longer.
    // At most 2^20: by then 1365 workgroups follow each other in each of the 768 places of 256 compute units, and a launch of 256 threads
    // each stays a factor of 16 below the 2^32 threads that it may hold.
    const long long steps = (rays.S + (PAIRS ? 31 : 63)) / (PAIRS ? 32 : 64);
    const long long fine = std::min(items * steps / (kWaves * 32) / 8 * 8, 1LL << 20);
    if (blocks < fine) blocks = fine;
    if (blocks > need) blocks = (need + 7) / 8 * 8;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kWaves * 64), kLdsBytes, stream, g, m, rays, out);
    return hipGetLastError();
}

template <int KIND, int C, int H, int NH, bool CC, int CG, int GT = LP_F32>
hipError_t launch_fwd(const GridDev& g, const MlpDev& m, const RaysDev& rays, const FwdOut& out, int n_cu,
                      hipStream_t stream)
{
    // as many workgroups as fit a compute unit's registers at least (see launch_items), a multiple of the 8 XCDs, no more than the rays need
    const long long blocks = (3LL * n_cu + 7) / 8 * 8;
    if constexpr (kPairs<KIND, C, CG>) {
        // Pairs where a SIMD has no more steps that way, and two waves for each SIMD remain unless a ray is one step either way.
        // 256 .. 44 000 rays x 24 .. 330 samples, eight structures and decoders, time in single rays over that in pairs: where
        // pairs are taken 0.97 .. 1.84 (330 samples: 0.96 .. 1.18; 24: up to 1.8), elsewhere 0.60 .. 1.24 (up to 2000 rays of more
        // than 64 samples 0.60 .. 1.08: fewer waves, each with more steps in a row).
        const long long simds = 4LL * n_cu, pair_items = (rays.M + 1) / 2;
        auto share = [&](long long items) { return (items + simds - 1) / simds; };
        const bool no_more = share(pair_items) * ((rays.S + 31) / 32) <= share(rays.M) * ((rays.S + 63) / 64);
        if (no_more && (rays.S <= 32 || pair_items >= 2 * simds))
            return launch_items<KIND, C, H, NH, CC, CG, GT, true>(g, m, rays, out, blocks, stream);
    }
    return launch_items<KIND, C, H, NH, CC, CG, GT, false>(g, m, rays, out, blocks, stream);
}

template <int KIND>
hipError_t dispatch_fwd(const GridDev& g, const MlpDev& m, const RaysDev& rays, const FwdOut& out, int n_cu,
                        hipStream_t stream)
{
    const int C = m.dims[0], CG = g.C, H = m.dims[1], NH = m.n_layers - 1;
    // grids stored in bf16 / fp16: plain inputs; the contraction is a run-time branch of these kernels
#define LP_CASE(c, h, nh)                                                                                     \
    if (C == c && CG == c && H == h && NH == nh && g.dtype != LP_F32)                  \
        return g.dtype == LP_BF16 ? launch_fwd<KIND, c, h, nh, false, c, LP_BF16>(g, m, rays, out, n_cu, stream) \
                                  : launch_fwd<KIND, c, h, nh, false, c, LP_F16>(g, m, rays, out, n_cu, stream);
    LP_CASE(16, 32, 1) LP_CASE(16, 64, 1) LP_CASE(32, 32, 1) LP_CASE(32, 64, 1)
    LP_CASE(16, 32, 2) LP_CASE(16, 64, 2) LP_CASE(32, 32, 2) LP_CASE(32, 64, 2)
#undef LP_CASE
    if (g.dtype != LP_F32 && CG == C) return hipErrorInvalidValue;   // (the decoder kernels read any storage type)
#define LP_CASE(c, cg, h, nh)                                                                          \
    if (C == c && CG == cg && H == h && NH == nh)                                                      \
        return g.contract > 0.0 ? launch_fwd<KIND, c, h, nh, true, cg>(g, m, rays, out, n_cu, stream) \
                                : launch_fwd<KIND, c, h, nh, false, cg>(g, m, rays, out, n_cu, stream);
    LP_CASE(16, 16, 32, 1) LP_CASE(16, 16, 64, 1) LP_CASE(32, 32, 32, 1) LP_CASE(32, 32, 64, 1)
    LP_CASE(16, 16, 32, 2) LP_CASE(16, 16, 64, 2) LP_CASE(32, 32, 32, 2) LP_CASE(32, 32, 64, 2)
#undef LP_CASE
    // 16 grid channels + direction inputs (the two-MLP decoder merged into one MLP of 32 inputs)
#define LP_CASE(h, nh)                                                                                  \
    if (C == 32 && CG == 16 && H == h && NH == nh)                                                      \
        return g.contract > 0.0 ? launch_fwd<KIND, 32, h, nh, true, 16, kAnyDtype>(g, m, rays, out, n_cu, stream) \
                                : launch_fwd<KIND, 32, h, nh, false, 16, kAnyDtype>(g, m, rays, out, n_cu, stream);
    LP_CASE(32, 1) LP_CASE(64, 1) LP_CASE(32, 2) LP_CASE(64, 2)
#undef LP_CASE
    return hipErrorInvalidValue;
}

// hash tables: the storage type and the contraction are run-time branches of one set of kernels
hipError_t dispatch_fwd_hash(const GridDev& g, const MlpDev& m, const RaysDev& rays, const FwdOut& out, int n_cu,
                             hipStream_t stream)
{
    const int C = m.dims[0], H = m.dims[1], NH = m.n_layers - 1;
#define LP_CASE(c, h, nh)                         \
    if (C == c && g.C == c && H == h && NH == nh) \
        return launch_fwd<LP_GRID_HASH, c, h, nh, false, c, kAnyDtype>(g, m, rays, out, n_cu, stream);
    LP_CASE(16, 32, 1) LP_CASE(16, 64, 1) LP_CASE(32, 32, 1) LP_CASE(32, 64, 1)
    LP_CASE(16, 32, 2) LP_CASE(16, 64, 2) LP_CASE(32, 32, 2) LP_CASE(32, 64, 2)
#undef LP_CASE
    // 16 table channels + direction inputs (the two-MLP decoder merged into one MLP of 32 inputs)
#define LP_CASE(h, nh)                             \
    if (C == 32 && g.C == 16 && H == h && NH == nh) \
        return launch_fwd<LP_GRID_HASH, 32, h, nh, false, 16, kAnyDtype>(g, m, rays, out, n_cu, stream);
    LP_CASE(32, 1) LP_CASE(64, 1) LP_CASE(32, 2) LP_CASE(64, 2)
#undef LP_CASE
    return hipErrorInvalidValue;
}

// HexPlanes: likewise one set of kernels
hipError_t dispatch_fwd_hexplane(const GridDev& g, const MlpDev& m, const RaysDev& rays, const FwdOut& out, int n_cu,
                                 hipStream_t stream)
{
    const int C = m.dims[0], H = m.dims[1], NH = m.n_layers - 1;
#define LP_CASE(c, h, nh)                         \
    if (C == c && g.C == c && H == h && NH == nh) \
        return launch_fwd<LP_GRID_HEXPLANE, c, h, nh, false, c, kAnyDtype>(g, m, rays, out, n_cu, stream);
    LP_CASE(16, 32, 1) LP_CASE(16, 64, 1) LP_CASE(32, 32, 1) LP_CASE(32, 64, 1)
    LP_CASE(16, 32, 2) LP_CASE(16, 64, 2) LP_CASE(32, 32, 2) LP_CASE(32, 64, 2)
#undef LP_CASE
    // 16 plane channels + direction inputs (the two-MLP decoder merged into one MLP of 32 inputs)
#define LP_CASE(h, nh)                             \
    if (C == 32 && g.C == 16 && H == h && NH == nh) \
        return launch_fwd<LP_GRID_HEXPLANE, 32, h, nh, false, 16, kAnyDtype>(g, m, rays, out, n_cu, stream);
    LP_CASE(32, 1) LP_CASE(64, 1) LP_CASE(32, 2) LP_CASE(64, 2)
#undef LP_CASE
    return hipErrorInvalidValue;
}

}  // namespace

bool mfma_supported(const GridDev& g, const MlpDev& m)
{
    if (g.kind != LP_GRID_VOXEL && g.kind != LP_GRID_TRIPLANE && g.kind != LP_GRID_HASH && g.kind != LP_GRID_HEXPLANE)
        return false;
    // inputs: all of them grid channels (16 or 32), or 16 grid channels + 16 direction inputs
    const bool plain = m.n_enc == 0 && m.dims[0] == g.C && (g.C == 16 || g.C == 32);
    const bool with_dir = m.n_enc > 0 && g.C == 16 && m.dims[0] == 32 && m.n_enc <= 16;
    if (!plain && !with_dir) return false;
        if (m.n_feat != 3 || m.dims[m.n_layers] != 4) return false;
    if (m.n_layers != 2 && m.n_layers != 3) return false;
    const int H = m.dims[1];
    if (H != 32 && H != 64) return false;
    if (m.n_layers == 3 && m.dims[2] != H) return false;
    // 32-bit byte offsets inside one scene's tensor (below 4 GiB), 16-byte aligned tensors
    const unsigned long long n0 = (unsigned long long)g.N[0], n1 = (unsigned long long)g.N[1], n2 = (unsigned long long)g.N[2];
    const unsigned long long per_scene = n0 * n1 * n2 * g.C;  // voxel tensor of one scene
    if (g.kind == LP_GRID_VOXEL) {
        if (per_scene >= (1ull << 30)) return false;
        if ((uintptr_t)g.data[0] & 15u) return false;
    } else if (g.kind == LP_GRID_HASH) {
        // a table whose size is a power of two (`mod size` is a mask in these kernels)
        const unsigned long long T = (unsigned long long)g.hash_size;
        if (T == 0 || (T & (T - 1)) != 0 || T * g.C >= (1ull << 30)) return false;
        if ((uintptr_t)g.data[0] & 15u) return false;
    } else {
        if (n0 * n1 * g.C >= (1ull << 30) || n1 * n2 * g.C >= (1ull << 30) || n2 * n0 * g.C >= (1ull << 30)) return false;
        for (int p = 0; p < 3; ++p)
            if ((uintptr_t)g.data[p] & 15u) return false;
        if (g.kind == LP_GRID_HEXPLANE) {   // the space-time planes under the same limits
            const unsigned long long nt = (unsigned long long)g.NT;
            if (n0 * nt * g.C >= (1ull << 30) || n1 * nt * g.C >= (1ull << 30) || n2 * nt * g.C >= (1ull << 30))
                return false;
            for (int p = 0; p < 3; ++p)
                if ((uintptr_t)g.data_t[p] & 15u) return false;
        }
    }
    return true;
}

hipError_t launch_fwd_mfma(const GridDev& g, const MlpDev& m, const RaysDev& rays, const FwdOut& out, int n_cu,
                           hipStream_t stream)
{
    if (g.kind == LP_GRID_HASH) return dispatch_fwd_hash(g, m, rays, out, n_cu, stream);
    if (g.kind == LP_GRID_HEXPLANE) return dispatch_fwd_hexplane(g, m, rays, out, n_cu, stream);
    return g.kind == LP_GRID_VOXEL ? dispatch_fwd<LP_GRID_VOXEL>(g, m, rays, out, n_cu, stream)
                                   : dispatch_fwd<LP_GRID_TRIPLANE>(g, m, rays, out, n_cu, stream);
}

}  // namespace lp
