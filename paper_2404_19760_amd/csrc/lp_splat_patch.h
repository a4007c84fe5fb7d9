// Patches of an image for the naive Splatter (Section 3.3 "Splatter"): 8 x 4 neighbouring pixels whose rays are marched
// together, eight points of each per step, and the weights of a step's points on the texels that they reach.
//
// Why patches: push and gradient are bound by the texels that a step touches (atomic adds, reads). 8 x 4 pixels share
// far more of them than pixels in a row. 160^3 voxels over [-2.75, 2.75]^3, 128^2 pixels at distance 2.5, 160 points a ray:
// a ray by itself reaches about 3 texels a point, four pixels of a row with eight points each 1.60, 8 x 4 pixels 0.60.
// The rays come as a list; the length of an image's row is found from their end points (lp_image_rows.h). It decides the order of
// the work only: whatever is found, every ray belongs to one patch, and a patch whose rays are not neighbours is taken
// apart by its caller.
#pragma once
#include "lp_image_rows.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_tile_lds.h"

namespace lp {

namespace {

constexpr int kPatchH = 4;           // lines of pixels of a patch
constexpr int kPatchPoints = 8;      // of a ray per step

// Patches of RAYS / 4 x 4 pixels of an image `row` wide and ceil(M / row) high, row after row of patches.
template <int RAYS>
struct PatchGrid {
    static constexpr int kW = RAYS / kPatchH;
    long long M, row, per_row, count;
    __device__ explicit PatchGrid(long long m, long long w) : M(m), row(w)
    {
        per_row = (w + kW - 1) / kW;
        count = per_row * (((m + w - 1) / w + kPatchH - 1) / kPatchH);
    }
    // first pixel of line y of patch p, and where that line ends (rays [first, end): none if the line does not exist)
    __device__ void line(long long p, int y, long long& first, long long& end) const
    {
        const long long x0 = p % per_row * kW, at = (p / per_row * kPatchH + y) * row;
        first = at + x0;
        end = min(min(at + row, first + kW), M);
    }
    // ray i of patch p (line i / kW) and whether it exists
    __device__ long long ray(long long p, int i, bool& ok) const
    {
        long long first, end;
        line(p, i / kW, first, end);
        const long long r = first + i % kW;
        ok = r < end;
        return min(r, M - 1);
    }
};

// ---- the texels of a step and the weights on them ----

// LDS of a wave: weights[slot][ray] (a slot is a texel that the step reaches), the slots' texel offsets in elements, and the
// slots of the window's texels; when the weights stand, that last part is the caller's.
template <int RAYS>
struct PatchLds {
    static constexpr int kSlots = RAYS == 32 ? 224 : 160;
    static constexpr int kRow = RAYS * 4 + 16;     // bytes of a slot's weights (16 of padding: no bank conflicts)
    static constexpr int kTexels = 1024;           // texels of a window at most, and bytes of the last part
    static constexpr int OFFSETS = kSlots * kRow;
    static constexpr int MAP = OFFSETS + kSlots * 4;
    static constexpr int kBytes = MAP + kTexels;
    static_assert(OFFSETS % 16 == 0 && MAP % 16 == 0 && kSlots <= 256, "16-byte accesses; a slot is a byte");
};

struct PatchCells {
    Cell3 c[kPatchPoints];
    unsigned there;   // a bit per point: the lane's ray has it
};

// extremes over the wave, whose upper half holds what its lower half holds
__device__ __forceinline__ int group_min(int v)
{
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true));
    return min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
}
__device__ __forceinline__ int group_max(int v) { return -group_min(-v); }

// Cells of points j0 .. of the lane's ray; `end`: first point that is not to be taken.
template <bool CC>
__device__ __forceinline__ PatchCells patch_cells(const GridDev& g, const RayGeom& q, bool ray_ok, int j0, int end, int S)
{
    PatchCells p;
    p.there = 0u;
#pragma unroll
    for (int k = 0; k < kPatchPoints; ++k) {
        p.c[k] = sample_cell<CC>(g, q, min(j0 + k, S - 1));
        p.there |= (ray_ok && j0 + k < end) ? 1u << k : 0u;
    }
    return p;
}

// Plane `pl` of the points [from, from + len) of every ray (`only` >= 0: of this one): the texels that they reach get slots, and
// weights[slot][ray] receives the sum of the ray's interpolation weights on the texel.  Number of slots; 0: no
// points; -1: too many texels.  A cell's corners are shared out to the lane groups of a ray (32 rays: by the slowest axis; 16: by
// the two slowest), so that no two lanes meet in a weight of one point.
template <int KIND, int C, int RAYS>
__device__ __forceinline__ int patch_weights(uint32_t area, const GridDev& g, const PatchCells& cells, int from, int len, int only,
                                             int pl, int lane)
{
    using L = PatchLds<RAYS>;
    constexpr bool kFlat = KIND == LP_GRID_TRIPLANE, kQuarter = RAYS == 16;
    const int ray = lane & (RAYS - 1), d0 = kQuarter ? lane >> 5 : lane / RAYS, d1_mine = (lane >> 4) & 1;
    constexpr int kFace = (kFlat ? 4 : 8) * RAYS / 64;   // corners of a lane
    const int a0 = kFlat ? pl : 0, a1 = kFlat ? (pl + 1) % 3 : 1;   // the plane's axes (uniform: no indexed registers)
    constexpr int a2 = 2;
    auto at = [](const int (&v)[3], int a) { return a == 0 ? v[0] : a == 1 ? v[1] : v[2]; };
    auto atf = [](const float (&v)[3], int a) { return a == 0 ? v[0] : a == 1 ? v[1] : v[2]; };
    const unsigned members = (only < 0 || ray == only) ? cells.there & (((1u << len) - 1u) << from) : 0u;
    if (__ballot(members != 0u) == 0ull) return 0;
    // (a ray's cells go one way along every axis: its extremes are at its first and last point)
    int lo[3], hi[3];
    {
        int first[3], last[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) first[a] = last[a] = 0;
#pragma unroll
        for (int k = 0; k < kPatchPoints; ++k) {
            const bool starts = k == from, ends = ((members >> k) & 1u) != 0u;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                first[a] = starts ? cells.c[k].i[a] : first[a];
                last[a] = ends ? cells.c[k].i[a] : last[a];
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = group_min(members ? min(first[a], last[a]) : 0x3fffffff);
            hi[a] = group_max(members ? max(first[a], last[a]) : -1);
        }
    }
    const int l0 = at(lo, a0), l1 = at(lo, a1), l2 = kFlat ? 0 : lo[a2];
    const int e0 = at(hi, a0) - l0 + 2, e1 = at(hi, a1) - l1 + 2, e2 = kFlat ? 1 : hi[a2] - l2 + 2;
    // (each factor first: the product of three sides of a large grid does not fit 32 bits)
    if (max(e0, max(e1, e2)) > L::kTexels || e0 * e1 > L::kTexels || e0 * e1 * e2 > L::kTexels) return -1;
    const int total = e0 * e1 * e2;
    // which texels
    wave_lds_fence();
    lds_put<u32x4>(area + L::MAP + 16 * lane, u32x4{0u, 0u, 0u, 0u});
    wave_lds_fence();
    // corner d of the lane: 0 or 1 along the plane's second axis and along the third
    auto along1 = [&](int d) { return kQuarter ? d1_mine : kFlat ? d : d >> 1; };
    auto along2 = [&](int d) { return kFlat ? 0 : d & 1; };
    int dense[kPatchPoints];   // the lane's first corner in the window
#pragma unroll
    for (int k = 0; k < kPatchPoints; ++k) {
        const Cell3& c = cells.c[k];
        dense[k] = ((at(c.i, a0) - l0 + d0) * e1 + at(c.i, a1) - l1 + along1(0)) * e2 + (kFlat ? 0 : c.i[a2] - l2);
        if ((members >> k) & 1u) {
            const uint8_t one = 1;
#pragma unroll
            for (int d = 0; d < kFace; ++d)
                lds_put<uint8_t>(area + L::MAP + dense[k] + (along1(d) - along1(0)) * e2 + along2(d), one);
        }
    }
    wave_lds_fence();
    int n_slots = 0;
    const float inv12 = __builtin_amdgcn_rcpf((float)(e1 * e2)), inv2 = __builtin_amdgcn_rcpf((float)e2);
    auto small_div = [](int n, float inv) { return (int)(((float)n + 0.5f) * inv); };   // (n < 2^12; one half keeps the rounding away)
    for (int n0 = 0; n0 < total; n0 += 64) {
        const int n = n0 + lane;
        const bool touched = lds_get<uint8_t>(area + L::MAP + n) != 0;
        const unsigned long long all = __ballot(touched);
        const int slot = n_slots + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)all, 0u));
        if (touched && slot < L::kSlots) {
            lds_put<uint8_t>(area + L::MAP + n, (uint8_t)slot);
            const int t0 = small_div(n, inv12), rest = n - t0 * (e1 * e2);
            const int t1 = kFlat ? rest : small_div(rest, inv2), t2 = kFlat ? 0 : rest - t1 * e2;
            unsigned off;
            if constexpr (KIND == LP_GRID_TRIPLANE)
                off = ((unsigned)(l0 + t0) * (unsigned)(a1 == 0 ? g.N[0] : a1 == 1 ? g.N[1] : g.N[2]) + (unsigned)(l1 + t1)) * C;
            else if constexpr (KIND == LP_GRID_HASH)   // (a table whose size is a power of two; colliding texels keep slots of their own)
                off = (((unsigned)(l0 + t0) ^ (unsigned)(l1 + t1) * 2654435761u ^ (unsigned)(l2 + t2) * 805459861u) & (g.hash_size - 1u)) * C;
            else
                off = (((unsigned)(l0 + t0) * (unsigned)g.N[1] + (unsigned)(l1 + t1)) * (unsigned)g.N[2] + (unsigned)(l2 + t2)) * C;
            lds_put<uint32_t>(area + L::OFFSETS + 4 * slot, off);
        }
        n_slots += __popcll(all);
    }
    if (n_slots > L::kSlots) return -1;
    for (int i = lane; i < n_slots * (L::kRow / 16); i += 64) lds_put<u32x4>(area + 16 * i, u32x4{0u, 0u, 0u, 0u});
    wave_lds_fence();
    // the weights: a lane adds to its own ray's column, point after point.  (The upper face of a point may be the lower one of the
    // next, which is another lane's: a fence between points.)
    const uint32_t column = area + 4 * ray;
    uint32_t where[kPatchPoints][kFace];
#pragma unroll
    for (int k = 0; k < kPatchPoints; ++k)
        if ((members >> k) & 1u) {
#pragma unroll
            for (int d = 0; d < kFace; ++d)
                where[k][d] = column + L::kRow * (uint32_t)lds_get<uint8_t>(area + L::MAP + dense[k] + (along1(d) - along1(0)) * e2 + along2(d));
        }
#pragma unroll
    for (int k = 0; k < kPatchPoints; ++k) {
        if ((members >> k) & 1u) {
            const Cell3& c = cells.c[k];
            const float w0 = d0 ? atf(c.f, a0) : atf(c.g, a0);
            float old[kFace];
#pragma unroll
            for (int d = 0; d < kFace; ++d) old[d] = lds_get<float>(where[k][d]);
#pragma unroll
            for (int d = 0; d < kFace; ++d) {
                float w = w0 * (along1(d) ? atf(c.f, a1) : atf(c.g, a1));
                if constexpr (!kFlat) w *= along2(d) ? c.f[a2] : c.g[a2];
                lds_put<float>(where[k][d], old[d] + w);
            }
        }
        wave_lds_fence();
    }
    return n_slots;
}

// Has `take(from, len, only)` take a step's points: all at once; where they reach too many texels (false) four, then one, then
// one of a single ray, which always fits.
template <int RAYS, class Take>
__device__ __forceinline__ void patch_steps(Take take)
{
    int from = 0, len = kPatchPoints, only = -1;
    while (from < kPatchPoints) {
        if (take(from, len, only)) {
            if (only >= 0 && ++only < RAYS) continue;
            only = -1;
            from += len;
            if (from % 4 == 0) len = 4;
        } else if (len > 1) {
            len = len > 4 ? 4 : 1;
        } else {
            only = 0;
        }
    }
}

// First texel of a scene in plane `pl`.
template <int KIND>
__device__ __forceinline__ size_t scene_texel(const GridDev& g, int pl, int scene)
{
    if constexpr (KIND == LP_GRID_TRIPLANE) return (size_t)scene * g.N[pl] * g.N[(pl + 1) % 3];
    else if constexpr (KIND == LP_GRID_HASH) return (size_t)scene * g.hash_size;
    else return (size_t)scene * g.N[0] * g.N[1] * g.N[2];
}

// How the lines of a patch are taken: in parts of consecutive lines, each marched as one.  Bit y: line y begins a part, as its
// rays do not lie near those of line y - 1 at both ends: the border of two views, mostly.  (However small the structure is: no
// bound on the whole of a patch that an image's need tells the two apart, and steps across a border go one point of one ray
// at a time: 20 such patches of 1400 took 2.0 of 2.2 ms, 2 x 157 x 139 rays x 237 points, 42 x 31 x 34 x 16 voxels.)
// Bit 4 + y: not all rays of line y near each other, in one scene and finite; its part goes ray by ray.
template <int RAYS, bool CC>
__device__ __forceinline__ unsigned patch_lines(const GridDev& g, const RayGeom& q, bool ok, int S, int lane)
{
    constexpr int kW = PatchGrid<RAYS>::kW, kNext = 5;   // kNext: texels between neighbours
    const float geometry[8] = {q.ox, q.oy, q.oz, q.dx, q.dy, q.dz, q.near, q.delta};
    float probe = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) probe = fmaf(geometry[i], 0.0f, probe);
    const Cell3 c0 = sample_cell<CC>(g, q, 0), c1 = sample_cell<CC>(g, q, S - 1);
    const unsigned long long oks = __ballot(ok);
    const int ray = lane & (RAYS - 1), left = ray % kW ? ray - 1 : ray, above = ray >= kW ? ray - kW : ray;
    auto apart_from = [&](int other) {   // (all lanes take part)
        int most = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a)
            most = max(most, max(abs(c0.i[a] - __shfl(c0.i[a], other, 64)), abs(c1.i[a] - __shfl(c1.i[a], other, 64))));
        const int scene = __shfl(q.scene, other, 64);
        return ((oks >> other) & 1ull) != 0ull && (most > kNext || scene != q.scene);
    };
    const bool from_above = apart_from(above), from_left = apart_from(left);
    const unsigned long long breaks = __ballot(ok && from_above), bad = __ballot(ok && (from_left || probe != 0.0f));
    unsigned lines = 1u;
#pragma unroll
    for (int y = 0; y < kPatchH; ++y) {
        const unsigned long long line = ((1ull << kW) - 1ull) << (y * kW);
        lines |= ((breaks & line) ? 1u << y : 0u) | ((bad & line) ? 16u << y : 0u);
    }
    return lines;
}

// Calls part(first line, line behind the last, whether its rays go one by one) for every part.
template <class Part>
__device__ __forceinline__ void patch_parts(unsigned lines, Part part)
{
    for (int y0 = 0; y0 < kPatchH;) {
        int y1 = y0 + 1;
        while (y1 < kPatchH && !((lines >> y1) & 1u)) ++y1;
        part(y0, y1, ((lines >> (4 + y0)) & ((1u << (y1 - y0)) - 1u)) != 0u);
        y0 = y1;
    }
}

}  // namespace

}  // namespace lp
