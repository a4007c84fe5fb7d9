// Sampling of the hash structure for the 32 samples of a step by the whole wavefront (Section 3.2).
//
// What bounds it: the address path of the vector memory unit. With one lane per sample, each 16-byte load of a
// wave touches up to 64 texels; a step of 32 samples on a 32-channel triplane then takes 10 300 cycles of a SIMD
// (three waves on it) whatever the locality, 3 800 when the lanes of a texel read its line together.  So the
// samples' corner weights and offsets are published in LDS, and the wave passes over the samples with the 8 (or 4,
// or 2) lanes of a texel side by side: every load instruction reads whole texels.  The interpolated channels are
// split into bf16 hi + lo and stored as an input image (lp_tile_lds.h), from where the matrix-core operands are
// read.
#pragma once
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_tile_lds.h"

namespace lp {

// One sample's record: corner weights, then offsets in elements. voxel: 8 weights (corner 4dx + 2dy + dz), offset of
// corner 0; triplane: 12 weights (plane p, corner 2da + db at 4p + ..), 3 offsets; hash table: 8 weights, 8 offsets.
// The stride keeps the records of neighbouring samples in different banks.
template <int KIND>
struct GatherRecord {
    static constexpr int kWeights = KIND == LP_GRID_TRIPLANE ? 12 : 8;
    static constexpr int kDwords = KIND == LP_GRID_VOXEL ? 12 : 20;
    static constexpr int kBytes = kDwords * 4;
    static constexpr int kStep = 32 * kBytes;   // of a step
};

// The record of this lane's sample (lane & 31) at cell c; the two lane groups share the work.
template <int KIND, int C>
__device__ __forceinline__ void publish_gather(uint32_t at, int lane, const GridDev& g, const Cell3& c)
{
    const int col = lane & 31, grp = lane >> 5;
    at += col * GatherRecord<KIND>::kBytes;
    if constexpr (KIND == LP_GRID_TRIPLANE) {
        // group 0: planes 0 and 2, group 1: plane 1 and the offsets
        const float a1 = grp ? c.f[1] : c.f[0], b1 = grp ? c.f[2] : c.f[1], a0 = 1.0f - a1, b0 = 1.0f - b1;
        lds_put<f32x4>(at + 16 * grp, f32x4{a0 * b0, a0 * b1, a1 * b0, a1 * b1});
        const float z1 = c.f[2], z0 = 1.0f - z1, x1 = c.f[0], x0 = 1.0f - x1;
        f32x4 v = {z0 * x0, z0 * x1, z1 * x0, z1 * x1};
        const uint32_t o0 = ((unsigned)c.i[0] * (unsigned)g.N[1] + (unsigned)c.i[1]) * C;
        const uint32_t o1 = ((unsigned)c.i[1] * (unsigned)g.N[2] + (unsigned)c.i[2]) * C;
        const uint32_t o2 = ((unsigned)c.i[2] * (unsigned)g.N[0] + (unsigned)c.i[0]) * C;
        v[0] = grp ? __uint_as_float(o0) : v[0];
        v[1] = grp ? __uint_as_float(o1) : v[1];
        v[2] = grp ? __uint_as_float(o2) : v[2];
        lds_put<f32x4>(at + 32 + 16 * grp, v);
    } else {
        // group g: the four corners of dx = g
        const float wx = grp ? c.f[0] : 1.0f - c.f[0];
        const float y1 = c.f[1], y0 = 1.0f - y1, z1 = c.f[2], z0 = 1.0f - z1;
        lds_put<f32x4>(at + 16 * grp, f32x4{wx * y0 * z0, wx * y0 * z1, wx * y1 * z0, wx * y1 * z1});
        if constexpr (KIND == LP_GRID_VOXEL) {
            lds_put<uint32_t>(at + 32, (((unsigned)c.i[0] * (unsigned)g.N[1] + (unsigned)c.i[1]) * (unsigned)g.N[2] +
                                        (unsigned)c.i[2]) * C);
        } else {
            const unsigned mask = g.hash_size - 1u;   // (a power of two in these kernels)
            const unsigned hx = (unsigned)c.i[0] + grp, hy = (unsigned)c.i[1] * 2654435761u, hz = (unsigned)c.i[2] * 805459861u;
            const unsigned hy1 = hy + 2654435761u, hz1 = hz + 805459861u;
            lds_put<u32x4>(at + 32 + 16 * grp, u32x4{((hx ^ hy ^ hz) & mask) * C, ((hx ^ hy ^ hz1) & mask) * C,
                                                     ((hx ^ hy1 ^ hz) & mask) * C, ((hx ^ hy1 ^ hz1) & mask) * C});
        }
    }
}

// Passes over the 32 samples whose records stand at `rec`: features into the image at `img` (hi, then lo).
// AHEAD: the loads of the next pass are issued before a pass is interpolated.
template <int KIND, int C, int GT, bool AHEAD = true>
struct WaveGather {
    using Rec = GatherRecord<KIND>;
    using Image = TileImage<C, false>;
    static constexpr unsigned kElem = GT == LP_F32 ? 4u : 2u;
    static constexpr int kLanes = C * kElem / 16;      // lanes of a texel
    static constexpr int kSamples = 64 / kLanes;       // samples of a pass (at most 32)
    static constexpr int kPasses = kSamples >= 32 ? 1 : 32 / kSamples;
    static constexpr int kVals = 16 / kElem;           // channels of a lane
    static constexpr int kCorners = Rec::kWeights;

    struct Raw {
        uint4 v[kCorners];
    };

    __device__ static __forceinline__ int sample_of(int lane, int pass) { return pass * kSamples + lane / kLanes; }

    __device__ static __forceinline__ void load(const GridDev& g, int scene, uint32_t rec, int lane, int pass, Raw& raw)
    {
        const uint32_t at = rec + sample_of(lane, pass) * Rec::kBytes;
        const uint32_t mine = (lane % kLanes) * 16;
        auto fetch = [](const char* p, uint32_t off) { return *reinterpret_cast<const uint4*>(p + off); };
        if constexpr (KIND == LP_GRID_TRIPLANE) {
            const u32x4 o = lds_get<u32x4>(at + 48);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
                const int a = pl, b = (pl + 1) % 3;
                const char* P = reinterpret_cast<const char*>(g.data[pl]) + (size_t)scene * g.N[a] * g.N[b] * C * kElem;
                const uint32_t off = o[pl] * kElem + mine;
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    raw.v[4 * pl + d] = fetch(P + (size_t)(((d >> 1) * (unsigned)g.N[b] + (d & 1)) * C * kElem), off);
            }
        } else if constexpr (KIND == LP_GRID_VOXEL) {
            const char* V = reinterpret_cast<const char*>(g.data[0]) + (size_t)scene * g.N[0] * g.N[1] * g.N[2] * C * kElem;
            const size_t sz = C * kElem, sy = g.N[2] * sz, sx = g.N[1] * sy;
            const uint32_t off = lds_get<uint32_t>(at + 32) * kElem + mine;
#pragma unroll
            for (int d = 0; d < 8; ++d) raw.v[d] = fetch(V + (d >> 2) * sx + ((d >> 1) & 1) * sy + (d & 1) * sz, off);
        } else {
            const char* V = reinterpret_cast<const char*>(g.data[0]) + (size_t)scene * g.hash_size * C * kElem;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 o = lds_get<u32x4>(at + 32 + 16 * h);
#pragma unroll
                for (int d = 0; d < 4; ++d) raw.v[4 * h + d] = fetch(V, o[d] * kElem + mine);
            }
        }
    }

    __device__ static __forceinline__ void finish(uint32_t rec, uint32_t img, int lane, int pass, const Raw& raw)
    {
        const int s = sample_of(lane, pass);
        const uint32_t at = rec + s * Rec::kBytes;
        float f[kVals];
#pragma unroll
        for (int e = 0; e < kVals; ++e) f[e] = 0.0f;
#pragma unroll
        for (int q = 0; q < kCorners / 4; ++q) {
            const f32x4 w = lds_get<f32x4>(at + 16 * q);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                float v[kVals];
                unpack_values<GT>(raw.v[4 * q + d], v);
#pragma unroll
                for (int e = 0; e < kVals; ++e) f[e] += w[d] * v[e];
            }
        }
        const int chunk = lane % kLanes;
        uint32_t hi[kVals / 2], lo[kVals / 2];
#pragma unroll
        for (int e = 0; e < kVals / 2; ++e) split2(f[2 * e], f[2 * e + 1], hi[e], lo[e]);
        if constexpr (kVals == 4) {   // half a chunk
            const uint32_t p = img + s * Image::kRow + (((chunk >> 1) ^ Image::swizzle(s)) << 4) + (chunk & 1) * 8;
            lds_put<u32x2>(p, u32x2{hi[0], hi[1]});
            lds_put<u32x2>(p + Image::bytes(32), u32x2{lo[0], lo[1]});
        } else {
            const uint32_t p = img + s * Image::kRow + ((chunk ^ Image::swizzle(s)) << 4);
            lds_put<u32x4>(p, u32x4{hi[0], hi[1], hi[2], hi[3]});
            lds_put<u32x4>(p + Image::bytes(32), u32x4{lo[0], lo[1], lo[2], lo[3]});
        }
    }

    __device__ static __forceinline__ void run(const GridDev& g, int scene, uint32_t rec, uint32_t img, int lane)
    {
        Raw raw[AHEAD && kPasses > 1 ? 2 : 1];
        load(g, scene, rec, lane, 0, raw[0]);
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            if constexpr (AHEAD && kPasses > 1) {
                if (p + 1 < kPasses) load(g, scene, rec, lane, p + 1, raw[(p + 1) & 1]);
                finish(rec, img, lane, p, raw[p & 1]);
            } else {
                finish(rec, img, lane, p, raw[0]);
                if (p + 1 < kPasses) load(g, scene, rec, lane, p + 1, raw[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// GT = kAnyDtype: the storage type is a uniform run-time branch
template <int KIND, int C, int GT, bool AHEAD = true>
__device__ __forceinline__ void wave_gather(const GridDev& g, int scene, uint32_t rec, uint32_t img, int lane)
{
    if constexpr (GT == kAnyDtype) {
        if (g.dtype == LP_F32) WaveGather<KIND, C, LP_F32, AHEAD>::run(g, scene, rec, img, lane);
        else if (g.dtype == LP_BF16) WaveGather<KIND, C, LP_BF16, AHEAD>::run(g, scene, rec, img, lane);
        else WaveGather<KIND, C, LP_F16, AHEAD>::run(g, scene, rec, img, lane);
    } else {
        WaveGather<KIND, C, GT, AHEAD>::run(g, scene, rec, img, lane);
    }
}

// The 32 samples of a step from the cell of each lane's sample to the layer-1 operands.
template <int KIND, int C, int GT, bool AHEAD = true>
__device__ __forceinline__ void wave_features(const GridDev& g, int scene, const Cell3& c, uint32_t rec, uint32_t img, int lane,
                                              Frag (&fh)[C / 16], Frag (&fl)[C / 16])
{
    using Image = TileImage<C, false>;
    publish_gather<KIND, C>(rec, lane, g, c);
    wave_lds_fence();   // (also: the last step's reads of the image are done)
    wave_gather<KIND, C, GT, AHEAD>(g, scene, rec, img, lane);
    wave_lds_fence();   // (also: the reads of the records are done)
    const uint32_t own = img + Image::own(lane);
#pragma unroll
    for (int s = 0; s < C / 16; ++s) {
        fh[s] = lds_chunk(own ^ Image::own_step(s));
        fl[s] = lds_chunk((own ^ Image::own_step(s)) + Image::bytes(32));
    }
}

// LDS bytes a wave needs for wave_features: records, then the image
template <int KIND, int C>
struct WaveGatherLds {
    static constexpr int IMG = GatherRecord<KIND>::kStep;
    static constexpr int kBytes = IMG + 2 * TileImage<C, false>::bytes(32);
    static_assert(IMG % 256 == 0, "an image starts at a multiple of its swizzled bits");
};

}  // namespace lp
