// Matrix-core backward kernel of the Renderer (Eq. (2), Section 3.4 of the paper) over neighbouring rays: a
// wavefront marches a PATCH of an image (four pixels each of two rows, four samples of each ray per 32-sample step), a TILE
// of a list (four consecutive rays, eight samples of each) or, where rays do not run side by side, one ray (32 samples),
// from the last samples to the first.
// A workgroup is eight wavefronts of 256 registers, two per SIMD, that share the MLP's weights in LDS: no wave waits for another
// between the staging of the weights and the final sums.  Each also publishes the number of its steps there, and the other wave of its SIMD reads
// it, as it is found: nothing but s_setprio may depend on it.
//
// Per step a wave
//   1. recomputes the MLP forward from the sampled features (nothing was stored but one scalar per ray),
//   2. rebuilds the transmittance from the cached optical depth and evaluates Eq. (2) with scans over
//      the samples of each ray,
//   3. back-propagates on the matrix cores: input gradients dX = W^T dZ chained in registers, weight
//      gradients dW = dZ X^T contracted over the samples of the step,
//   4. adds the feature gradient to the grid gradient: scatter_step below, as matrix products over small windows of
//      texels or, where the step's samples are too far apart for it, with the run-merging walk of lp_mfma_bwd_common.h.
//
// What bounds it and why it is laid out like this (256^3 x 16 voxels, 800^2 rays x 512 samples, and eight
// 256^2 x 32 triplanes, 4 x 256^2 rays x 192 samples each):
//   - The grid gradient is bound by the rate of atomic adds (2.1e10 64-byte lines/s on this chip, whatever
//     the locality). One ray's samples touch 3.1 (voxel) and 9.9 (triplane) lines per sample after run
//     merging; the union of the texels that four neighbouring rays touch with eight samples each is 0.70 and
//     3.63 lines per sample, of a patch with four samples each 0.52 and 2.56 (counted), and the scatter's matrix products shrink
//     alike.  (Patches against tiles, a whole training step: eight triplanes 115.7 -> 107.6 ms, one triplane 128^2 x 32, 128^2 rays,
//     735 -> 665 us, 256^3 x 16 voxels 61.1 -> 60.7 ms, a hash table 460 -> 451 us.)
//   - A wave does not overlap its own vector and matrix instructions; two waves per SIMD do. The
//     accumulators of the weight gradients (94 registers for 16-64-64-4: the two thin matrices on 16 x 16
//     and 4 x 4 tiles) leave room for two waves only if a step's activations live in LDS instead of registers.
//     Per SIMD the voxel kernel issues vector instructions in 52 % of the cycles and keeps the matrix cores busy in
//     39 %, the triplane kernel 45 % and 38 % (1315 and 1634 vector instructions a step; 46.4 and 82.1 ms a launch).
//   - In LDS they are transposed by the reads (lp_tile_lds.h); on the matrix cores the transposition by 0/1
//     products took 36 of the 168 products of a step and as many permutes. The transposed weights of the
//     input-gradient chain are column reads of the same images, which halves the LDS that weights take.
//   - Vector work alternates with products that do not wait for it (weave below).
//   - Products with four rows (the output layer) carry the hi and the lo halves of the operand in rows
//     that would be empty, or in empty parts of the K range: 8 instead of 12 in the forward, 2 instead of 6 in the
//     input-gradient chain.  The weight gradient takes 24 products of sixteen 4 x 4 blocks instead of 12 of 32 x 32.
#pragma once
#include "lp_image_rows.h"
#include "lp_kernels.h"
#include "lp_mfma.h"
#include "lp_mfma_mlp.h"
#include "lp_mfma_bwd_common.h"
#include "lp_tile_lds.h"
#include "lp_tile_scatter.h"
#include "lp_weave.h"

namespace lp {

namespace {

constexpr int kTileWaves = 8;
// A patch: four neighbouring pixels each of two rows of an image, four samples of each ray per step.
constexpr int kPatchRays = 8, kPatchSamples = 4, kLogPatchSamples = 2, kLogTileSamples = 3;
static_assert((1 << kLogPatchSamples) == kPatchSamples && (1 << kLogTileSamples) == kTileSamples && kPatchRays * kPatchSamples == 32);
// From pixel to pixel at most, in the middle of the rays.  Images of 96^2 to 256^2 pixels, 16 and 32 channels, 64 to 512 samples; time of the
// backward in tiles over that in patches, mean (least, largest), by pixel distance, where from 0.7 on more and more patches fall apart
// into tiles and from 1 on into single rays:
//              0.6    0.7 .. 0.85         0.9 .. 1.0          1.02 .. 1.1         1.2                  1.33 .. 1.5
//   voxels 16  1.19   0.99 (0.86, 1.23)   0.99 (0.90, 1.11)   1.02 (0.96, 1.12)   1.00 (0.98, 1.06)    0.99 (0.93, 1.06)
//   voxels 32  1.35   1.05 (0.98, 1.32)   1.03 (1.00, 1.10)   1.02 (0.97, 1.06)   1.01 (0.98, 1.03)    1.00 (0.95, 1.01)
//   planes     1.23   1.06 (0.90, 1.32)   1.06 (1.00, 1.17)   1.03 (0.98, 1.10)   1.01 (0.97, 1.05)    1.00 (0.94, 1.06)
//   hash       1.21   1.00 (0.88, 1.18)   1.01 (0.95, 1.08)   1.04 (0.99, 1.07)   1.02 (1.00, 1.05)    1.00 (0.97, 1.07)
// Behind the lines nothing is gained on average, and images of voxels took up to 1.08 times as long in patches.  (The least at 0.7 to 1.0: 128^2 pixels x 64
// samples, one item to a wave, some of them single rays; four items to a wave, 1.00 .. 1.2.)
template <int KIND>
constexpr double kPixelTexels = KIND == LP_GRID_VOXEL ? 1.3 : 1.5;

// LDS in bytes: the waves' step tensors first (so that a wave's base has none of the address bits that the
// images' exclusive-ors flip), then the weights, then the waves' small areas.
template <int C, int H, int NH>
struct TileLds {
    using W1 = TileImage<C, false>;
    using WH = TileImage<H, true>;
    // one wave: two tensors of 32 samples, each a hi and a lo image
    static constexpr int kAct = 8192;
    static constexpr int A = 0, B = kAct;
    static constexpr int W2_AT = kTileWaves * 2 * kAct;
    static constexpr int W1_AT = W2_AT + (NH == 2 ? 2 * WH::bytes(H) : 0);
    static constexpr int kWo = 2 * H + 16;                       // bytes of an output-layer row (padded)
    static constexpr int WO_AT = W1_AT + 2 * W1::bytes(H);       // 4 rows hi, 4 rows lo
    static constexpr int BIAS_AT = WO_AT + 8 * kWo;              // b1[H] b2[H] bo[4]
    static constexpr int SMALL_AT = BIAS_AT + (2 * H + 4) * 4;
    // one wave: output gradients; per ray of a step, fp64, the optical depth up to the step's end and the sum over later steps
    static constexpr int SUMS = 512;
    static constexpr int kSmall = SUMS + kPatchRays * 16;
    static constexpr int STEPS_AT = SMALL_AT + kTileWaves * kSmall;   // steps that each wave has done
    static constexpr int kTotal = STEPS_AT + kTileWaves * 4;
    static_assert(W2_AT % 4096 == 0 && W1_AT % 1024 == 0 && SMALL_AT % 16 == 0 && kSmall % 16 == 0, "alignment");
    static_assert(kTotal <= 160 * 1024, "LDS budget of a gfx950 compute unit");
};

// All of the wave's loads have arrived.  For loads whose values only some lanes use: the others' way around that use leaves
// them outstanding to the compiler, and whatever next takes their registers then waits, in every turn of a loop, for all memory
// operations issued since.
__device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// Inclusive prefix sum over the samples of a ray: segments of 4 or 8 lanes, or (`alone`) of 32.  k = position in
// the segment.
__device__ __forceinline__ float ray_scan(float v, int k, bool alone)
{
    float t = dpp_or_zero<0x111, 0xf>(v);
    v += k >= 1 ? t : 0.0f;
    t = dpp_or_zero<0x112, 0xf>(v);
    v += k >= 2 ? t : 0.0f;
    t = dpp_or_zero<0x114, 0xf>(v);
    v += k >= 4 ? t : 0.0f;
    t = dpp_or_zero<0x118, 0xf>(v);
    v += alone ? t : 0.0f;
    t = dpp_or_zero<0x142, 0xa>(v);
    v += alone ? t : 0.0f;
    return v;
}

// Interpolated channels [ch0, ch0 + NCH) at cell c: the corners in groups of four (the two x faces of a voxel
// cell, the planes of a triplane); a group's loads are issued together.  STAGED: one group after the
// other (at most 4 NCH registers of raw texels), else the compiler may issue them all.
template <int KIND, int C, int NCH, int GT, bool STAGED>
__device__ __forceinline__ void gather_stream(const GridDev& g, int scene, const Cell3& c, int ch0, float* feat)
{
    constexpr int kPerVec = GT == LP_F32 ? 4 : 8, kVecs = NCH / kPerVec;
    constexpr unsigned kElem = GT == LP_F32 ? 4u : 2u;
    constexpr int kGroups = KIND == LP_GRID_TRIPLANE ? 3 : 2;
#pragma unroll
    for (int k = 0; k < NCH; ++k) feat[k] = 0.0f;
#pragma unroll
    for (int gr = 0; gr < kGroups; ++gr) {
        uint4 raw[4][kVecs];
        float w[4];
        // (a uniform pointer per corner and one byte offset per lane, below 4 GiB: no address arithmetic per load)
        if constexpr (KIND == LP_GRID_TRIPLANE) {
            const int a = gr, b = (gr + 1) % 3;
            const char* P = reinterpret_cast<const char*>(g.data[gr]) + (size_t)scene * g.N[a] * g.N[b] * C * kElem;
            const unsigned off = (((unsigned)c.i[a] * (unsigned)g.N[b] + (unsigned)c.i[b]) * C + ch0) * kElem;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int da = d >> 1, db = d & 1;
                const char* p = P + ((size_t)da * g.N[b] + db) * C * kElem;
#pragma unroll
                for (int i = 0; i < kVecs; ++i) raw[d][i] = *reinterpret_cast<const uint4*>(p + off + 16 * i);
                w[d] = (da ? c.f[a] : 1.0f - c.f[a]) * (db ? c.f[b] : 1.0f - c.f[b]);
            }
        } else if constexpr (KIND == LP_GRID_HASH) {
            const char* V = reinterpret_cast<const char*>(g.data[0]) + (size_t)scene * g.hash_size * C * kElem;
            unsigned slot[8];
            hash_corner_slots(c, g.hash_size, slot);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int dy = d >> 1, dz = d & 1;
                const unsigned off = (slot[4 * gr + d] * C + ch0) * kElem;
#pragma unroll
                for (int i = 0; i < kVecs; ++i) raw[d][i] = *reinterpret_cast<const uint4*>(V + off + 16 * i);
                w[d] = (gr ? c.f[0] : 1.0f - c.f[0]) * (dy ? c.f[1] : 1.0f - c.f[1]) * (dz ? c.f[2] : 1.0f - c.f[2]);
            }
        } else {
            const char* V = reinterpret_cast<const char*>(g.data[0]) +
                            (size_t)scene * g.N[0] * g.N[1] * g.N[2] * C * kElem;
            const size_t sz = C * kElem, sy = g.N[2] * sz, sx = g.N[1] * sy;
            const unsigned off = ((((unsigned)c.i[0] * (unsigned)g.N[1] + (unsigned)c.i[1]) * (unsigned)g.N[2] + (unsigned)c.i[2]) * C + ch0) * kElem;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int dy = d >> 1, dz = d & 1;
                const char* p = V + gr * sx + dy * sy + dz * sz;
#pragma unroll
                for (int i = 0; i < kVecs; ++i) raw[d][i] = *reinterpret_cast<const uint4*>(p + off + 16 * i);
                w[d] = (gr ? c.f[0] : 1.0f - c.f[0]) * (dy ? c.f[1] : 1.0f - c.f[1]) * (dz ? c.f[2] : 1.0f - c.f[2]);
            }
        }
        if constexpr (STAGED) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int i = 0; i < kVecs; ++i) {
                float v[kPerVec];
                unpack_values<GT>(raw[d][i], v);
#pragma unroll
                for (int e = 0; e < kPerVec; ++e) feat[kPerVec * i + e] += w[d] * v[e];
            }
        if constexpr (STAGED) __builtin_amdgcn_sched_barrier(0);
    }
}

// One launch's work items: patches (four pixels each of two rows of an image), consecutive tiles of kTileRays rays, or single
// rays.  As many rounds as leave no wave of any workgroup without an item hand them out: in groups of kTileWaves, the workgroups of a
// round at places scrambled by `group_mul` (neighbouring rays add into the same lines; spread over time their adds do not queue up at one
// L2 channel), and from round to round a workgroup moves by `shift` places, or it would meet the same columns of an image again and again.
// A group is eight neighbours, or (`spread`) one item of each eighth of the list.  Items cost unlike amounts, by where their rays
// lie: with eight neighbouring patches to a workgroup and the places in their order in short lists, the dearest workgroup took 1.28 times the
// mean of 160^3 x 32 voxels in contract coordinates (256^2 rays, four rounds), now a step of training takes 6.6 instead of 8.3 ms; eight
// triplanes 107.8 -> 107.0, the others alike.  Tiles are spread in contract coordinates only (150^2 to 300^2 pixels, seven shapes each, of
// neighbours 0.95 to 1.02 times the speed): elsewhere neighbours share more than the spread evens out (150^2 pixels x 48 samples, 90^3
// voxels and planes, 1.17 times the speed of the spread, 16-32-4 1.25; 181^2 to 300^2 pixels 1.00 to 1.03), and so do single rays (32^2 to
// 140^2 pixels, 64 to 400 samples, 1.00 to 1.02).  What is left goes to the first
// `busy` waves of a workgroup, to as many workgroups as that takes: up to four of them have a SIMD each, where a ray takes 0.55 to 0.7 of the time beside
// another.  (2600 rays in random order x 480 samples, 96^3 x 16 voxels, 16-64-64-4: the last 552 rays on 69 full workgroups 303 us,
// spread over all 243; 32-64-64-4 on triplanes 128^2 469 -> 400.)
enum class Items { kRays, kTiles, kPatches };   // kPatches: if the rays are found to be an image's, else tiles
struct TileSchedule {
    long long rounds, group_mul, group_step[2];
    int shift;
    int busy, tail_per_xcd;   // (tail_per_xcd: workgroups of an XCD that the last, partial round reaches)
    Items items;
};

// Int: long long, or unsigned on the device (items below 2^31)
template <class Int>
__host__ __device__ inline TileSchedule tile_schedule(Items kind, Int items, Int blocks)
{
    TileSchedule sc;
    sc.items = kind;
    const Int waves = blocks * (Int)kTileWaves, rounds = items / waves, tail = items - rounds * waves;
    Int busy = (tail + blocks - 1) / blocks;
    if (rounds && busy > (Int)(kTileWaves / 2)) busy = (Int)kTileWaves;   // (they share SIMDs anyhow: 5128 tiles, 679 -> 669 us)
    sc.rounds = (long long)rounds;
    sc.busy = (int)busy;
    sc.tail_per_xcd = busy ? (int)(((tail + busy - 1) / busy + 7) / 8) : 0;
    // multiplier of the scramble: a prime that does not divide the number of groups, so that
    // group -> group * mul mod n_groups is a bijection
    const Int n_groups = rounds * blocks;
    Int mul = 1;
    for (Int p : {(Int)7919, (Int)7907, (Int)7901, (Int)7883})
        if (n_groups % p != 0) { mul = p; break; }
    sc.group_mul = (long long)mul;
    sc.shift = (int)(blocks * 5 / 8 | 1);
    for (int wraps = 0; wraps < 2; ++wraps)
        sc.group_step[wraps] = n_groups ? (long long)((sc.shift + (wraps ? 0 : blocks)) * mul % n_groups) : 0;
    return sc;
}

// Steps of the longest wave.
template <class Int>
__host__ __device__ inline Int wave_steps(Int items, Int blocks, Int samples, Int step)
{
    const Int waves = blocks * (Int)kTileWaves;
    return (items + waves - 1) / waves * ((samples + step - 1) / step);
}

template <int KIND, int C, int H, int NH, bool CC, int GT>
__global__ __launch_bounds__(kTileWaves * 64) void bwd_tile_kernel(GridDev g, MlpDev m, RaysDev rays, BwdIo io,
                                                                   TileSchedule sched)
{
    using L = TileLds<C, H, NH>;
    using IW1 = typename L::W1;      // also the image of a step's input features
    using IH = typename L::WH;       // also the image of a step's hidden tensors
    constexpr int MB = H / 32, KS1 = C / 16, KSH = H / 16, G16 = H / 16;
    constexpr int kLoH = IH::bytes(32), kLoF = IW1::bytes(32);   // hi image -> lo image of a step's tensors
    extern __shared__ uint4 lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LdsByte*)reinterpret_cast<char*>(lds_raw);

    // ---- staging ----
    if constexpr (NH == 2) stage_image<IH, H, true>(lds + L::W2_AT, m.W[1], H, H);
    stage_image<IW1, C, false>(lds + L::W1_AT, m.W[0], H, C);
    for (int idx = threadIdx.x; idx < 4 * (H / 8); idx += blockDim.x) {   // output layer, rows
        const int row = idx / (H / 8), chunk = idx % (H / 8);
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = m.W[NH][row * H + 16 * (chunk >> 1) + 8 * (e / 4) + 4 * (chunk & 1) + (e % 4)];
        Frag hi, lo;
        split8(x, hi, lo);
        lds_put_chunk(lds + L::WO_AT + row * L::kWo + chunk * 16, hi);
        lds_put_chunk(lds + L::WO_AT + (4 + row) * L::kWo + chunk * 16, lo);
    }
    float* bias = reinterpret_cast<float*>(reinterpret_cast<char*>(lds_raw) + L::BIAS_AT);
    for (int i = threadIdx.x; i < H; i += blockDim.x) {
        bias[i] = m.b[0][i];
        bias[H + i] = NH == 2 ? m.b[1][i] : 0.0f;
    }
    if (threadIdx.x < 4) bias[2 * H + threadIdx.x] = m.b[NH][threadIdx.x];
    if (threadIdx.x < kTileWaves) lds_put<int>(lds + L::STEPS_AT + 4 * threadIdx.x, 0);
    __syncthreads();

    uint32_t lane_id = threadIdx.x & 63;   // (refreshed like the addresses)
    const int lane = lane_id, col = lane & 31, grp = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t acts = lds + wave * 2 * L::kAct;               // this wave's step tensors
    const uint32_t dz_at = lds + L::SMALL_AT + wave * L::kSmall;  // its output gradients
    const int S = rays.S;

    // gradient accumulators, alive for the whole kernel
    f32x16 dW2[MB][MB];                    // NH == 2
    f32x16 dW1w[MB];                       // C == 32
    f32x4 dW1t[G16];                       // C == 16
    f32x4 dWo = {0.0f, 0.0f, 0.0f, 0.0f};  // lane = hidden feature (H = 32: twice, for half of the samples each), register = output
    float db1[C == 32 ? MB : G16], db2[MB];
    float dbo[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int a = 0; a < MB; ++a) {
        db2[a] = 0.0f;
        if constexpr (C == 32) { dW1w[a] = zero16(); db1[a] = 0.0f; }
#pragma unroll
        for (int b = 0; b < MB; ++b)
            if constexpr (NH == 2) dW2[a][b] = zero16();
    }
#pragma unroll
    for (int a = 0; a < G16; ++a) {
        const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (C == 16) { dW1t[a] = z; db1[a] = 0.0f; }
    }

    // ---- work items ----
    // (the rays' pixels must share texels for a patch to be worth it, see kPixelTexels)
    int row = 0, per_row = 0;   // of the image: pixels, patches
    if (sched.items == Items::kPatches) {
        row = __builtin_amdgcn_readfirstlane((int)find_row(g, rays, kPixelTexels<KIND>, 1e30, *reinterpret_cast<int*>(lds_raw)));
        sched.items = Items::kTiles;
        if (row) {
            const unsigned lines = ((unsigned)rays.M + row - 1) / row;
            per_row = (row + kTileRays - 1) / kTileRays;
            const unsigned n_patches = per_row * ((lines + 1) / 2), n_tiles = ((unsigned)rays.M + kTileRays - 1) / kTileRays;
            // (rows that are no multiple of four leave places empty)
            if (20 * wave_steps<unsigned>(n_patches, gridDim.x, S, kPatchSamples) <= 21 * wave_steps<unsigned>(n_tiles, gridDim.x, S, kTileSamples))
                sched = tile_schedule<unsigned>(Items::kPatches, n_patches, gridDim.x);
        }
    }
    const Items items = sched.items;
    const bool spread = items == Items::kPatches || (items == Items::kTiles && g.contract > 0.0);   // (see TileSchedule)
    const int xcd = blockIdx.x % 8, at = blockIdx.x / 8;
    const long long n_groups = sched.rounds * gridDim.x;   // of the whole rounds
    int left = (int)sched.rounds;                          // rounds to come; -1: the partial one is over too
    int place = blockIdx.x;                                // of the workgroup in the round
    long long group = left ? (place * sched.group_mul) % n_groups : 0, item = 0;
    // rays [first, end) of line y of the item (a patch has two lines, another item one; none: first >= end)
    auto line = [&](int y, long long& first, long long& end) {
        if (items == Items::kPatches) {
            const unsigned p = (unsigned)item, l = 2 * (p / (unsigned)per_row) + y, x = p % (unsigned)per_row * kTileRays;
            first = (long long)l * row + x;
            end = min(min(first + kTileRays, ((long long)l + 1) * row), rays.M);
        } else {
            first = items == Items::kTiles ? item * kTileRays : item;
            end = y ? first : min(first + (items == Items::kTiles ? kTileRays : 1), rays.M);
        }
    };
    auto next_item = [&]() {   // false: none left
        if (left > 0) {
            item = spread ? wave * n_groups + group : group * kTileWaves + wave;
            place += sched.shift;
            const bool wraps = place >= (int)gridDim.x;
            if (wraps) place -= (int)gridDim.x;
            group += wraps ? sched.group_step[1] : sched.group_step[0];
            if (group >= n_groups) group -= n_groups;
            --left;
            return true;
        }
        if (left < 0) return false;
        left = -1;
        item = n_groups * kTileWaves + ((long long)sched.tail_per_xcd * xcd + at) * sched.busy + wave;
        if (wave >= sched.busy || at >= sched.tail_per_xcd) return false;
        long long first, end;
        line(0, first, end);
        return first < rays.M;
    };
    bool live = next_item();

    // the rays being marched, from number `sub` of the item on (four to a line): 2^(5 - log_samples) of them, 2^log_samples samples of each
    // per step.  (The lane's columns: ray col >> log_samples, sample col & (2^log_samples - 1).)
    int log_samples = 5, sub = 0, j0 = 0, scene = 0;
    auto step_sample = [&]() { return (int)lane_id & ((1 << log_samples) - 1); };   // this lane's sample in the step
    bool ray_ok = false;        // the lane's ray exists
    // What a step needs of its rays, 16 floats each, in two registers of the wave: value v of ray r in lane 8 r + v % 8 of
    // register v / 8.  (LDS has no room for eight rays beside the weights of 32-64-64-4.)
    int ray_data[2] = {0, 0};
    enum { kOrigin = 0, kDir = 3, kNear = 6, kDelta = 7, kDelta64 = 8, kDelta64Hi = 9, kThrough = 10, kUpstream = 11, kUpstreamDepth = 14 };
    // Values from number FROM on.  A single ray's are uniform and come by scalar reads: 16 reads across the lanes a step had taken the place of
    // four of LDS.  (Backward, 98 lists of random rays, voxels, planes and hash tables: 0.9 % less time; triplane 96^2 x 16, 4096 rays x 256
    // samples, 16-32-32-4: 170 -> 164 us, as before the change; images the same within 0.2 %.)
    auto ray_values = [&](auto from, auto& out) {
        constexpr int FROM = decltype(from)::value, N = sizeof(out) / sizeof(out[0]);
        if (log_samples == 5) {
#pragma unroll
            for (int i = 0; i < N; ++i) out[i] = __builtin_amdgcn_readlane(ray_data[(FROM + i) / 8], (FROM + i) % 8);
        } else {
            const int at = (((int)lane_id & 31) >> log_samples) * 32;
#pragma unroll
            for (int i = 0; i < N; ++i) out[i] = __builtin_amdgcn_ds_bpermute(at + (FROM + i) % 8 * 4, ray_data[(FROM + i) / 8]);
        }
    };
    // Optical depth up to the end of the current step, and the sum of w_j a_j over all later steps (fp64: see Eq. (2) below).  The
    // widest kernels have no registers left for them: in scratch memory they would be read behind the last step's atomic adds
    // (triplane 128^2 x 32, 16 384 rays x 77 samples: 350 us of backward with the depth in LDS, 366 in registers; 64^3 x 32 voxels under
    // 32-64-4: 9.86 ms a step in LDS, 9.66 in registers).
    constexpr bool kSumsInLds = C == 32 && H == 64 && NH == 2;
    typedef __attribute__((__vector_size__(2 * sizeof(double)))) double f64x2;
    double tau_end = 0.0, carry = 0.0;
    Cell3 cell;
    Frag fh[KS1], fl[KS1];

    auto geometry = [&]() {
        int v[kDelta64Hi + 1];
        ray_values(std::integral_constant<int, kOrigin>(), v);
        RayGeom q;
        q.ox = __int_as_float(v[kOrigin]); q.oy = __int_as_float(v[kOrigin + 1]); q.oz = __int_as_float(v[kOrigin + 2]);
        q.dx = __int_as_float(v[kDir]); q.dy = __int_as_float(v[kDir + 1]); q.dz = __int_as_float(v[kDir + 2]);
        q.near = __int_as_float(v[kNear]); q.delta = 0.0f;
        q.delta64 = __hiloint2double(v[kDelta64Hi], v[kDelta64]);
        q.scene = scene;
        q.time = 0.0f;
        return q;
    };
    // Loads the rays from `sub` on: a whole patch, a line of a patch or a tile, if they run side by side, else one.
    auto load_rays = [&]() {
        const int col = lane_id & 31, grp = lane_id >> 5;
        long long first, end;
        line(sub >> 2, first, end);
        first += sub & 3;
        const long long there = min(first, rays.M - 1);   // (behind an image's last line a patch may hold no ray)
        auto cell_of = [&](const RayGeom& q, int j) { return sample_cell_for<CC, GT>(g, q, j); };
        // the lane's ray of a patch
        auto patch_ray = [&](bool& ok) {
            long long first, end;
            line((col >> kLogPatchSamples) >> 2, first, end);
            const long long r = first + ((col >> kLogPatchSamples) & 3);
            ok = r < end;
            return r;
        };
        bool patch = false;
        if (items == Items::kPatches && sub == 0) {
            bool ok;
            const long long r = patch_ray(ok);
            patch = side_by_side(rays, ok ? r : there, cell_of);
        }
        bool tile = false;
        if (items != Items::kRays && !patch && (sub & 3) == 0) tile = side_by_side(rays, min(first + col / kTileSamples, end - 1), cell_of);
        log_samples = patch ? kLogPatchSamples : tile ? kLogTileSamples : 5;
        long long r = first + (tile ? col / kTileSamples : 0);
        ray_ok = r < end;
        if (patch) r = patch_ray(ray_ok);
        const long long ray = ray_ok ? r : there;
        const RayGeom q = load_ray_geom(rays, ray);
        scene = __builtin_amdgcn_readfirstlane(q.scene);
        const int k = step_sample();
        const float p0 = io.d_rgb[3 * ray + 0], p1 = io.d_rgb[3 * ray + 1], p2 = io.d_rgb[3 * ray + 2];
        const float p_alpha = io.d_alpha ? io.d_alpha[ray] : 0.0f;
        const float p_depth = io.d_depth ? io.d_depth[ray] : 0.0f;
        const float tau_S = io.cache[ray];
        // d(loss)/dT_S through alpha = 1 - T_S and rgb += T_S bg, times T_S
        const float kS = __expf(-tau_S) * (p_alpha - (p0 * io.bg[0] + p1 * io.bg[1] + p2 * io.bg[2]));
        // through the wave's LDS (nothing of a step is in it here) into the registers
        wave_lds_fence();
        if (k == 0 && grp == 0) {
            const uint32_t p = acts + L::B + (col >> log_samples) * 32;
            lds_put<f32x4>(p, f32x4{q.ox, q.oy, q.oz, q.dx});
            lds_put<f32x4>(p + 16, f32x4{q.dy, q.dz, q.near, q.delta});
            lds_put<double>(p + 256, q.delta64);
            lds_put<float>(p + 264, kS);
            lds_put<float>(p + 268, p0);
            lds_put<f32x4>(p + 272, f32x4{p1, p2, p_depth, 0.0f});
            if constexpr (kSumsInLds) lds_put<f64x2>(dz_at + L::SUMS + (col >> log_samples) * 16, f64x2{(double)tau_S, 0.0});
        }
        wave_lds_fence();
        ray_data[0] = lds_get<int>(acts + L::B + 4 * lane_id);
        ray_data[1] = lds_get<int>(acts + L::B + 256 + 4 * lane_id);
        wave_lds_fence();   // (the first rays are read right in front of a step, whose activations go to the same bytes)
        loads_done();
        tau_end = (double)tau_S;
        carry = 0.0;
        j0 = ((S - 1) >> log_samples) << log_samples;
    };
    // features of the lane's sample of the step at j0
    auto sample = [&]() {
        refresh(lane_id);
        const int grp = lane_id >> 5;
        const RayGeom q = geometry();
        cell = sample_cell_for<CC, GT>(g, q, min(j0 + step_sample(), S - 1));
        float feat[C / 2];
        gather_stream<KIND, C, C / 2, GT, (C == 32 || KIND == LP_GRID_TRIPLANE)>(g, scene, cell, grp * (C / 2), feat);
#pragma unroll
        for (int s = 0; s < KS1; ++s) split8(feat + 8 * s, fh[s], fl[s]);
        // complete before the scatter: memory operations return in order, and the scatter's adds are slow
#pragma unroll
        for (int s = 0; s < KS1; ++s)
#pragma unroll
            for (int w = 0; w < 4; ++w) asm volatile("" : "+v"(fh[s].d[w]), "+v"(fl[s].d[w]));
    };
    if (live) {
        load_rays();
        sample();
    }

    // addresses: this lane's chunks and columns of the step tensors; those of the weights differ by uniform amounts
    uint32_t own_h = acts + IH::own(lane), col_h = acts + IH::col32(lane), col16_h = acts + IH::col16(lane);
    uint32_t col64_h = acts + IH::col64(lane), own_f = acts + IW1::own(lane);
    uint32_t col_f = acts + (C == 32 ? IW1::col32(lane) : IW1::col16(lane)), col_f32 = acts + IW1::col32(lane);
    const uint32_t to_w2 = lds + L::W2_AT - acts, to_w1 = lds + L::W1_AT - acts;

    // Values 2 u, 2 u + 1 (u = 0 .. 7) of row block mb of a layer's output -> relu -> operand of the next layer, and
    // with every fourth pair a chunk into the images at `where`.
    auto activate_pair = [&](const f32x16& d, int mb, int u, uint32_t where, Frag (&h)[1][KSH], Frag (&l)[1][KSH]) {
        const int s = 2 * mb + u / 4;
        split2(relu_f(d[2 * u]), relu_f(d[2 * u + 1]), h[0][s].d[u % 4], l[0][s].d[u % 4]);
        pin(h[0][s].d[u % 4]);
        pin(l[0][s].d[u % 4]);
        if (u % 4 == 3) {
            lds_put_chunk((own_h ^ IH::own_step(s)) + where, h[0][s]);
            lds_put_chunk((own_h ^ IH::own_step(s)) + where + kLoH, l[0][s]);
        }
    };
    // The same for a gradient with the mask relu'(.) taken from the stored activation's hi half: 0 or 1 per half
    // (written out, or the compiler takes the halves apart), applied by 16-bit products on the split halves (left to
    // the compiler, which keeps the wait states between a vector write and a matrix read).
    auto gradient_pair = [&](const f32x16& d, int mb, int u, const Frag (&act)[2], Frag (&h)[1][KSH], Frag (&l)[1][KSH]) {
        typedef __attribute__((__vector_size__(4))) unsigned short u16x2;
        constexpr uint32_t kOnes = 0x00010001u;
        const int s = 2 * mb + u / 4;
        uint32_t on, hi, lo;
        split2(d[2 * u], d[2 * u + 1], hi, lo);
        asm("v_pk_min_u16 %0, %1, %2" : "=v"(on) : "v"(act[u / 4].d[u % 4]), "s"(kOnes));
        h[0][s].d[u % 4] = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, hi) * __builtin_bit_cast(u16x2, on)));
        l[0][s].d[u % 4] = __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, lo) * __builtin_bit_cast(u16x2, on)));
        pin(h[0][s].d[u % 4]);
        pin(l[0][s].d[u % 4]);
    };
    auto read_acts = [&](uint32_t where, int mb, Frag (&act)[2]) {
#pragma unroll
        for (int s = 0; s < 2; ++s) act[s] = lds_chunk((own_h ^ IH::own_step(2 * mb + s)) + where);
    };
    // D registers of a layer -> operand fragments -> the wave's images at A or B
    auto store_hidden = [&](uint32_t where, const Frag (&h)[1][KSH], const Frag (&l)[1][KSH]) {
#pragma unroll
        for (int s = 0; s < KSH; ++s) {
            lds_put_chunk((own_h ^ IH::own_step(s)) + where, h[0][s]);
            lds_put_chunk((own_h ^ IH::own_step(s)) + where + kLoH, l[0][s]);
        }
    };
    // (A wave with an item of the partial round starts an item behind the others: it is to be done when they are.  2559 rays in
    // random order x 445 samples, 16-32-32-4, a step of training: 201.7 -> 194.8 us; 6072 x 341, hash table of 32 channels, 507 -> 489.)
    int n_steps = 0;
    if (wave < sched.busy && at < sched.tail_per_xcd) {
        const int step = items == Items::kPatches ? kPatchSamples : items == Items::kTiles ? kTileSamples : 32;
        n_steps = -((S + step - 1) / step);
    }
    // The staging's loads too: a lane without a share of the weights passes by their use, and the kernels of one or two hidden layers of 32 waited
    // at the top of every step, and so for the adds of the step before.  (Backward, 2559 rays in random order x 445 samples through voxels, 16-32-32-4:
    // 169.4 -> 163.4 us, 16-32-4 139.5 -> 135.9, a hash table 171.3 -> 165.0.)
    loads_done();
    while (live) {
        refresh(own_h); refresh(own_f); refresh(lane_id);
        // Waves w and w + 4 share a SIMD, which serves the older one first: left alone, waves 0 .. 3 were done after 0.91 of the
        // time and 4 .. 7, alone by then, after 1.10 (four configurations within 0.02).  So the one behind goes first: 256^3 x 16
        // voxels 47.0 -> 43.9 ms, 64^3 x 32 voxels 6.9 -> 6.65, eight triplanes 80.3 -> 77.5.  (A word of LDS, read as it is found:
        // the order of the work changes, not the work.  Single rays gain too: 4096 in random order x 256 samples 243.7 -> 238.5 us a step of
        // training, 6144 x 128 on 32 channels 257 -> 253.)
        lds_put<int>(lds + L::STEPS_AT + 4 * wave, ++n_steps);
        const int partner_steps = lds_get<int>(lds + L::STEPS_AT + 4 * (wave ^ 4));   // (looked at where what was read behind it has arrived anyhow)
        const uint32_t own_w = own_h + to_w2, own_w1 = own_f + to_w1;
        const int lane = lane_id, col = lane & 31, grp = lane >> 5;
        // ---- MLP forward ----
        float z[4];
        {
            auto none = [](auto) {};
            Frag hh[1][KSH], hl[1][KSH], wh[2], wl[2];   // weights of two products, the next one's read ahead
            f32x16 acc[MB], acc2[MB];
            auto start = [&](f32x16 (&a)[MB], const float* b) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = *reinterpret_cast<const f32x4*>(b + 32 * mb + 8 * q + 4 * grp);
#pragma unroll
                        for (int p = 0; p < 4; ++p) a[mb][4 * q + p] = v[p];
                    }
            };
            auto read_w = [&](int slot, uint32_t at, int lo) { wh[slot] = lds_chunk(at); wl[slot] = lds_chunk(at + lo); };
            // product number i of the first layer: K-step i / 3 % KS1 of row block i / (3 KS1)
            auto w1_at = [&](int t) { return (own_w1 ^ IW1::own_step(t % KS1)) + (t / KS1) * 32 * IW1::kRow; };
            auto layer1 = [&](auto ic) {
                constexpr int i = decltype(ic)::value, t = i / 3, s = t % KS1, mb = t / KS1;
                if constexpr (i % 3 == 0 && t + 1 < MB * KS1) read_w((t + 1) & 1, w1_at(t + 1), IW1::bytes(H));
                acc[mb] = mfma1(i % 3 == 0 ? wl[t & 1] : wh[t & 1], i % 3 == 1 ? fl[s] : fh[s], acc[mb]);
                pin(acc[mb]);
            };
            start(acc, bias);
            read_w(0, w1_at(0), IW1::bytes(H));
            auto activate_1a = [&](auto u) { activate_pair(acc[0], 0, u, L::A, hh, hl); };
            {
                auto first = [&](auto i) { layer1(i); };
                weave<3 * KS1, 0, 0>(first, none);
            }
            if (__builtin_amdgcn_readfirstlane(partner_steps) > n_steps) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
            // second layer: the K-steps of the first block of activations for all rows, then those of the second block
            constexpr int T2 = MB * KSH;   // (row block, K-step) pairs in this order
            auto mb_of = [](int t) { return MB == 1 ? 0 : t < 4 ? t & 1 : (t - 4) >> 1; };
            auto s_of = [](int t) { return MB == 1 ? t : t < 4 ? t >> 1 : 2 + (t & 1); };
            auto w2_at = [&](int t) { return (own_w ^ IH::own_step(s_of(t))) + mb_of(t) * 32 * IH::kRow; };
            auto layer2 = [&](auto ic) {
                constexpr int i = decltype(ic)::value, t = i / 3;
                const int s = s_of(t), mb = mb_of(t);
                if constexpr (i % 3 == 0 && t + 1 < T2) read_w((t + 1) & 1, w2_at(t + 1), IH::bytes(H));
                acc2[mb] = mfma1(i % 3 == 0 ? wl[t & 1] : wh[t & 1], i % 3 == 1 ? hl[0][s] : hh[0][s], acc2[mb]);
                pin(acc2[mb]);
            };
            if constexpr (MB == 2) {
                auto second = [&](auto i) { layer1(std::integral_constant<int, decltype(i)::value + 3 * KS1>()); };
                weave<3 * KS1, 8, 1>(second, activate_1a);
            } else {
                repeat<0, 8>(activate_1a);
            }
            auto activate_1b = [&](auto u) { if constexpr (MB == 2) activate_pair(acc[MB - 1], MB - 1, u, L::A, hh, hl); };
            if constexpr (NH == 2) {
                start(acc2, bias + H);
                read_w(0, w2_at(0), IH::bytes(H));
                auto part1 = [&](auto i) { layer2(i); };
                weave<(MB == 2 ? 12 : 6), (MB == 2 ? 8 : 0), 2>(part1, activate_1b);
                if constexpr (MB == 2) {
                    auto part2 = [&](auto i) { layer2(std::integral_constant<int, decltype(i)::value + 12>()); };
                    weave<6, 0, 0>(part2, none);
                }
            } else {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc2[mb] = acc[mb];
            }
            // output layer: rows 0..3 and 4..7 of the operand are the hi halves of the four rows (one copy per
            // lane group), rows 8..11 and 12..15 their lo halves
            constexpr int kHere = NH == 2 ? L::B : L::A;
            f32x16 o;
            const f32x4 b = *reinterpret_cast<const f32x4*>(bias + 2 * H);
#pragma unroll
            for (int r = 0; r < 16; ++r) o[r] = r < 4 ? b[r] : 0.0f;
            const uint32_t wo_at = lds + L::WO_AT + ((col & 3) + ((col >> 1) & 4)) * L::kWo + grp * 16;
            Frag wo[2];
            wo[0] = lds_chunk(wo_at);
            auto output = [&](auto ic) {
                constexpr int i = decltype(ic)::value, s = i / 2;
                if constexpr (i % 2 == 0 && s + 1 < KSH) wo[(s + 1) & 1] = lds_chunk(wo_at + 32 * (s + 1));
                o = mfma1(wo[s & 1], i % 2 ? hh[0][s] : hl[0][s], o);
                pin(o);
            };
            auto activate_2a = [&](auto u) { if constexpr (NH == 2) activate_pair(acc2[0], 0, u, kHere, hh, hl); };
            auto activate_2b = [&](auto u) {
                if constexpr (NH == 2 && MB == 2) activate_pair(acc2[MB - 1], MB - 1, u, kHere, hh, hl);
                else activate_1b(u);
            };
            if constexpr (NH == 2 && MB == 2) {
                auto part3 = [&](auto i) { layer2(std::integral_constant<int, decltype(i)::value + 18>()); };
                weave<6, 8, 1>(part3, activate_2a);
            } else if constexpr (NH == 2) {
                repeat<0, 8>(activate_2a);
            }
            weave<4, (MB == 2 ? 8 : 0), 0>(output, activate_2b);
            if constexpr (MB == 2) {
                auto rest = [&](auto i) { output(std::integral_constant<int, decltype(i)::value + 4>()); };
                weave<4, 0, 0>(rest, none);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] = o[i] + o[4 + i];
        }

        // ---- Eq. (2); column col stands for sample j0 + k of the lane's ray (both lane groups alike) ----
        uint32_t zh0, zl0, zh1, zl1;
        {
            int v[kUpstreamDepth + 1 - kNear];
            ray_values(std::integral_constant<int, kNear>(), v);
            const float near = __int_as_float(v[0]), delta = __int_as_float(v[kDelta - kNear]), kS = __int_as_float(v[kThrough - kNear]);
            const float p0 = __int_as_float(v[kUpstream - kNear]), p1 = __int_as_float(v[kUpstream + 1 - kNear]), p2 = __int_as_float(v[kUpstream + 2 - kNear]);
            const float p_depth = __int_as_float(v[kUpstreamDepth - kNear]);
            const int k = step_sample(), j = j0 + k;
            const bool valid = ray_ok && j < S, alone = log_samples == 5;
            const int last = lane | ((1 << log_samples) - 1);
            const float t = near + ((float)j + 0.5f) * delta;
            // softplus and its derivative from one exponential
            const float ez = __expf(-fabsf(z[0])), rz = recip(1.0f + ez);
            const float sd = valid ? (fmaxf(z[0], 0.0f) + __logf(1.0f + ez)) * delta : 0.0f;
            const float incl = ray_scan(sd, k, alone);
            // (in fp64: a step of eight samples takes four times the subtractions of one of 32, and in fp32 each of them
            // rounds to the spacing of the whole depth, which at the front of an opaque ray is all of its weight; so does the sum over
            // later steps: summed in fp32 over 4096 samples, a patch's gradient of a ray whose terms cancel was 2.7 times as far from 64 bits as
            // a single ray's)
            const uint32_t sums_at = dz_at + L::SUMS + (col >> log_samples) * 16;
            if constexpr (kSumsInLds) {
                const f64x2 sums = lds_get<f64x2>(sums_at);
                tau_end = sums[0];
                carry = sums[1];
            }
            tau_end -= (double)__shfl(incl, last, 64);
            const float tau_start = (float)tau_end;
            const float Tprev = __expf(-(tau_start + (incl - sd)));
            const float w = Tprev * one_minus_exp_neg(sd);
            const float Tq = Tprev - w;
            const float c1 = recip(1.0f + __expf(-z[1])), c2 = recip(1.0f + __expf(-z[2])), c3 = recip(1.0f + __expf(-z[3]));
            const float aa = p0 * c1 + p1 * c2 + p2 * c3 + p_depth * t;
            const float wa = w * aa;
            const float pre = ray_scan(wa, k, alone);
            const float wa_total = __shfl(pre, last, 64);
            const float suf = wa_total - pre + wa;
            const float dsigma = delta * (Tq * aa - (suf - wa + (float)carry) + kS);
            carry += (double)wa_total;
            float dz[4];
            dz[0] = valid ? dsigma * (z[0] >= 0.0f ? rz : ez * rz) : 0.0f;
            dz[1] = valid ? w * p0 * c1 * (1.0f - c1) : 0.0f;
            dz[2] = valid ? w * p1 * c2 * (1.0f - c2) : 0.0f;
            dz[3] = valid ? w * p2 * c3 * (1.0f - c3) : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) dbo[i] += dz[i];
            split2(dz[0], dz[1], zh0, zl0);
            split2(dz[2], dz[3], zh1, zl1);
            lds_put<u32x4>(dz_at + col * 16, u32x4{zh0, zh1, zl0, zl1});   // (both lane groups the same)
            wave_lds_fence();   // the activations, the output gradients; every lane has read its ray's sums
            if (kSumsInLds && k == 0 && grp == 0) lds_put<f64x2>(sums_at, f64x2{tau_end, carry});
        }
        __builtin_amdgcn_sched_barrier(0);

        constexpr int kLast = NH == 2 ? L::B : L::A;   // the last hidden layer's activations
        refresh(own_h); refresh(col_h); refresh(col64_h);
        auto none = [](auto) {};
        // ---- last hidden layer: dZ = relu'(.) * (Wout^T dZo); the K range holds hi*hi, hi*lo, lo*hi ----
        f32x16 acc[MB];
        Frag gz_h[1][KSH], gz_l[1][KSH], act[MB][2];
        {
            Frag b;
            b.d[0] = zh0; b.d[1] = zh1; b.d[2] = grp ? 0u : zl0; b.d[3] = grp ? 0u : zl1;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                read_acts(kLast, mb, act[mb]);
                // columns 32 mb + (lane & 31) of the output layer's rows: hi halves for lane group 0, lo halves for 1
                const int t16 = lane & 15, c4 = t16 & 3, G = 2 * mb + ((lane >> 4) & 1);
                Frag a;
                lds_read_tr(lds + L::WO_AT + (4 * grp + (t16 >> 2)) * L::kWo + (2 * G + (c4 & 1)) * 16 + (c4 >> 1) * 8, a.d[0], a.d[1]);
                a.d[2] = grp ? 0u : a.d[0]; a.d[3] = grp ? 0u : a.d[1];
                acc[mb] = mfma1(a, b, zero16());
            }
        }
        // ---- dWo += dZo Hlast^T, beside the masking and splitting: sixteen 4 x 4 blocks (four outputs, four
        //      features), four samples per product ----
        {
            const int t16 = lane & 15;
            const uint32_t zp = dz_at + ((H == 32 ? 16 * (lane >> 5) : 0) + (t16 >> 2)) * 16;
            s16x4 ah[2], al[2], bh[2], bl[2];
            auto read = [&](int n) {
                const uint32_t hp = col64_h ^ IH::rows4(n & 3);
                ah[n & 1] = lds_tr(zp + n * 64); al[n & 1] = lds_tr(zp + n * 64 + 8);
                bh[n & 1] = lds_tr(hp + (n >> 2) * 16 * IH::kRow + kLast);
                bl[n & 1] = lds_tr(hp + (n >> 2) * 16 * IH::kRow + kLast + kLoH);
            };
            auto product = [&](auto ic) {
                constexpr int i = decltype(ic)::value, n = i / 3;
                if constexpr (i % 3 == 0 && n + 1 < H / 8) read(n + 1);
                dWo = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(i % 3 == 0 ? al[n & 1] : ah[n & 1], i % 3 == 1 ? bl[n & 1] : bh[n & 1], dWo, 0, 0, 0);
                pin(dWo);
            };
            auto piece = [&](auto ic) {
                constexpr int u = decltype(ic)::value;
                gradient_pair(acc[u / 8], u / 8, u % 8, act[u / 8], gz_h, gz_l);
            };
            read(0);
            weave<3 * H / 8, 8 * MB, 3>(product, piece);
        }

        if constexpr (NH == 2) {
            wave_lds_fence();   // the last layer's activations have been read
            store_hidden(L::B, gz_h, gz_l);
            refresh(own_h); refresh(col_h);
            const uint32_t col_w = col_h + to_w2;
            // ---- W2^T dZ2, row block after row block; beside it the transposed dZ2, db2 and the first block of dZ1 ----
            f32x16 up[MB];   // W2^T dZ2
            Frag g1_h[1][KSH], g1_l[1][KSH];
            {
                Frag wh[2], wl[2];
                auto read_w = [&](int t) {
                    wh[t & 1] = IH::read(col_w ^ (64 * (t / KSH)), (t % KSH) * 16 * IH::kRow);
                    wl[t & 1] = IH::read(col_w ^ (64 * (t / KSH)), (t % KSH) * 16 * IH::kRow + IH::bytes(H));
                };
                auto product = [&](auto ic) {
                    constexpr int i = decltype(ic)::value, t = i / 3, mb = t / KSH, s = t % KSH;
                    if constexpr (i % 3 == 0 && t + 1 < MB * KSH) read_w(t + 1);
                    up[mb] = mfma1(i % 3 == 0 ? wl[t & 1] : wh[t & 1], i % 3 == 1 ? gz_l[0][s] : gz_h[0][s],
                                   i == 3 * KSH * mb ? zero16() : up[mb]);
                    pin(up[mb]);
                };
                read_w(0);
                weave<3 * KSH, 0, 0>(product, none);
                if constexpr (MB == 2) {
                    read_acts(L::A, 0, act[0]);
                    auto second = [&](auto i) { product(std::integral_constant<int, decltype(i)::value + 3 * KSH>()); };
                    auto piece = [&](auto u) { gradient_pair(up[0], 0, u, act[0], g1_h, g1_l); };
                    weave<3 * KSH, 8, 2>(second, piece);
                }
            }
            wave_lds_fence();   // dZ2
            // ---- dW2 += dZ2 H1^T ; db2 += sum dZ2; beside it the last block of dZ1 ----
            {
                Frag ah[2], al[2], bh[2], bl[2];
                auto read_a = [&](int q) {   // (mb, ks) = q / 2, q % 2
                    ah[q & 1] = IH::read(col_h ^ (64 * (q / 2)), (q % 2) * 16 * IH::kRow + L::B);
                    al[q & 1] = IH::read(col_h ^ (64 * (q / 2)), (q % 2) * 16 * IH::kRow + L::B + kLoH);
                };
                auto read_b = [&](int t) {   // t = (mb, ks, nb)
                    const int nb = t % MB, ks = (t / MB) % 2;
                    bh[t & 1] = IH::read(col_h ^ (64 * nb), ks * 16 * IH::kRow + L::A);
                    bl[t & 1] = IH::read(col_h ^ (64 * nb), ks * 16 * IH::kRow + L::A + kLoH);
                };
                auto product = [&](auto ic) {
                    constexpr int i = decltype(ic)::value, t = i / 3, nb = t % MB, q = t / MB, mb = q / 2;
                    if constexpr (i % 3 == 0 && t + 1 < 2 * MB * MB) read_b(t + 1);
                    if constexpr (i % 3 == 0 && nb == 0 && q + 1 < 2 * MB) read_a(q + 1);
                    dW2[mb][nb] = mfma1(i % 3 == 0 ? al[q & 1] : ah[q & 1], i % 3 == 1 ? bl[t & 1] : bh[t & 1], dW2[mb][nb]);
                    pin(dW2[mb][nb]);
                    if constexpr (i % (3 * MB) == 1) {
                        db2[mb] = frag_sum(al[q & 1], frag_sum(ah[q & 1], db2[mb]));
                        pin(db2[mb]);
                    }
                };
                auto piece = [&](auto u) { gradient_pair(up[MB - 1], MB - 1, u, act[MB - 1], g1_h, g1_l); };
                read_acts(L::A, MB - 1, act[MB - 1]);
                read_a(0);
                read_b(0);
                weave<6 * MB * MB, 8, 1>(product, piece);
            }
#pragma unroll
            for (int s = 0; s < KSH; ++s) { gz_h[0][s] = g1_h[0][s]; gz_l[0][s] = g1_l[0][s]; }
        }
        // dZ1 and the features as images: NH == 2 in A and B, NH == 1 in B and A
        constexpr int kZ = NH == 2 ? L::A : L::B, kF = NH == 2 ? L::B : L::A;
        refresh(own_h); refresh(own_f); refresh(C == 32 ? col_f : col_f32);
        const uint32_t col_w1 = (C == 32 ? col_f : col_f32) + to_w1;
        wave_lds_fence();   // what they replace has been read
        store_hidden(kZ, gz_h, gz_l);
#pragma unroll
        for (int s = 0; s < KS1; ++s) {
            lds_put_chunk((own_f ^ IW1::own_step(s)) + kF, fh[s]);
            lds_put_chunk((own_f ^ IW1::own_step(s)) + kF + kLoF, fl[s]);
        }
        // ---- feature gradient, transposed: dF^T[sample][channel] = dZ1^T W1 (lane = channel) ----
        f32x16 dFt;
        {
            Frag wh[2], wl[2];
            auto read_w = [&](int s) {
                wh[s & 1] = IW1::read(col_w1, s * 16 * IW1::kRow);
                wl[s & 1] = IW1::read(col_w1, s * 16 * IW1::kRow + IW1::bytes(H));
            };
            auto product = [&](auto ic) {
                constexpr int i = decltype(ic)::value, s = i / 3;
                if constexpr (i % 3 == 0 && s + 1 < KSH) read_w(s + 1);
                dFt = mfma1(i % 3 == 0 ? gz_l[0][s] : gz_h[0][s], i % 3 == 1 ? wl[s & 1] : wh[s & 1], i == 0 ? zero16() : dFt);
                pin(dFt);
            };
            read_w(0);
            weave<3 * KSH, 0, 0>(product, none);
        }
        refresh(col_h); refresh(col16_h); refresh(col_f);
        wave_lds_fence();   // dZ1 and the features
        // ---- dW1 += dZ1 F^T ; db1 += sum dZ1 ----
        if constexpr (C == 32) {
            Frag bh[2], bl[2], ah[2], al[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                bh[ks] = IW1::read(col_f, ks * 16 * IW1::kRow + kF);
                bl[ks] = IW1::read(col_f, ks * 16 * IW1::kRow + kF + kLoF);
            }
            auto read_a = [&](int q) {
                ah[q & 1] = IH::read(col_h ^ (64 * (q / 2)), (q % 2) * 16 * IH::kRow + kZ);
                al[q & 1] = IH::read(col_h ^ (64 * (q / 2)), (q % 2) * 16 * IH::kRow + kZ + kLoH);
            };
            auto product = [&](auto ic) {
                constexpr int i = decltype(ic)::value, q = i / 3, mb = q / 2, ks = q % 2;
                if constexpr (i % 3 == 0 && q + 1 < 2 * MB) read_a(q + 1);
                dW1w[mb] = mfma1(i % 3 == 0 ? al[q & 1] : ah[q & 1], i % 3 == 1 ? bl[ks] : bh[ks], dW1w[mb]);
                pin(dW1w[mb]);
                if constexpr (i % 3 == 1) {
                    db1[mb] = frag_sum(al[q & 1], frag_sum(ah[q & 1], db1[mb]));
                    pin(db1[mb]);
                }
            };
            read_a(0);
            weave<6 * MB, 0, 0>(product, none);
        } else {
            const Frag bh = IW1::read(col_f, kF), bl = IW1::read(col_f, kF + kLoF);
            Frag ah[2], al[2];
            auto read_a = [&](int G) {
                ah[G & 1] = IH::read(col16_h ^ (32 * G), kZ);
                al[G & 1] = IH::read(col16_h ^ (32 * G), kZ + kLoH);
            };
            auto product = [&](auto ic) {
                constexpr int i = decltype(ic)::value, G = i / 3;
                if constexpr (i % 3 == 0 && G + 1 < G16) read_a(G + 1);
                dW1t[G] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(i % 3 == 0 ? al[G & 1] : ah[G & 1]), as_bf16x8(i % 3 == 1 ? bl : bh), dW1t[G], 0, 0, 0);
                pin(dW1t[G]);
                if constexpr (i % 3 == 1) {
                    db1[G] = frag_sum(al[G & 1], frag_sum(ah[G & 1], db1[G]));
                    pin(db1[G]);
                }
            };
            read_a(0);
            weave<3 * G16, 0, 0>(product, none);
        }
        __builtin_amdgcn_sched_barrier(0);

        // ---- features of the next step, then the scatter of this one ----
        const Cell3 here = cell;
        const int here_scene = scene;
        const int here_samples = 1 << log_samples;
        j0 -= here_samples;
        if (j0 < 0) {
            // the item's next ray that has not been marched: on the same line, or the first of the next one
            long long first, end;
            sub += 32 >> log_samples;
            line(sub >> 2, first, end);
            if ((sub & 3) && first + (sub & 3) >= end) {
                sub = (sub | 3) + 1;
                line(sub >> 2, first, end);
            }
            if (items == Items::kRays || sub >= (items == Items::kPatches ? kPatchRays : kTileRays) || first >= end) {
                sub = 0;
                live = next_item();
            }
            if (live) load_rays();
        }
        if (live) sample();
        __builtin_amdgcn_sched_barrier(0);
        refresh(lane_id);
        scatter_step<KIND, C>(g, io.d_grid, here_scene, acts + L::A, reinterpret_cast<char*>(lds_raw) + wave * 2 * L::kAct,
                              here, dFt, lane_id, here_samples);
        wave_lds_fence();
    }

    // ---- sums over the workgroup's waves (halving), then one record ----
    constexpr int kRegs = (NH == 2 ? 16 * MB * MB : 0) + (C == 32 ? 16 * MB : 4 * G16) + 4 + (C == 32 ? MB : G16) + MB + 4;
    static_assert(kTileWaves / 2 * kRegs * 256 <= L::kTotal, "half the waves' accumulators fit the LDS");
    auto each = [&](auto f) {
        int n = 0;
        if constexpr (NH == 2) {
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < MB; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) { float v = dW2[a][b][r]; f(n++, v); dW2[a][b][r] = v; }
        }
        if constexpr (C == 32) {
#pragma unroll
            for (int a = 0; a < MB; ++a) {
#pragma unroll
                for (int r = 0; r < 16; ++r) { float v = dW1w[a][r]; f(n++, v); dW1w[a][r] = v; }
                f(n++, db1[a]);
            }
        } else {
#pragma unroll
            for (int a = 0; a < G16; ++a) {
#pragma unroll
                for (int r = 0; r < 4; ++r) { float v = dW1t[a][r]; f(n++, v); dW1t[a][r] = v; }
                f(n++, db1[a]);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) { float v = dWo[r]; f(n++, v); dWo[r] = v; }
#pragma unroll
        for (int a = 0; a < MB; ++a) f(n++, db2[a]);
#pragma unroll
        for (int i = 0; i < 4; ++i) f(n++, dbo[i]);
    };
    float* sums = reinterpret_cast<float*>(lds_raw);
#pragma unroll 1
    for (int half = kTileWaves / 2; half >= 1; half >>= 1) {
        __syncthreads();
        if (wave >= half && wave < 2 * half) {
            float* mine = sums + (size_t)(wave - half) * kRegs * 64 + lane;
            each([&](int n, float& v) { mine[n * 64] = v; });
        }
        __syncthreads();
        if (wave < half) {
            const float* theirs = sums + (size_t)wave * kRegs * 64 + lane;
            each([&](int n, float& v) { v += theirs[n * 64]; });
        }
    }
    if (wave != 0) return;
    float* rec = io.ws + (size_t)blockIdx.x * io.ws_stride;
    if constexpr (NH == 2) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int nb = 0; nb < MB; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) rec[m.w_off[1] + (32 * mb + d_row(r, grp)) * H + 32 * nb + col] = dW2[mb][nb][r];
            const float s2 = db2[mb] + __shfl_xor(db2[mb], 32, 64);
            if (grp == 0) rec[m.b_off[1] + 32 * mb + col] = s2;
        }
    }
    const int i16 = lane & 15, q16 = lane >> 4;
    if constexpr (C == 32) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) rec[m.w_off[0] + (32 * mb + d_row(r, grp)) * C + col] = dW1w[mb][r];
            const float s1 = db1[mb] + __shfl_xor(db1[mb], 32, 64);
            if (grp == 0) rec[m.b_off[0] + 32 * mb + col] = s1;
        }
    } else {
#pragma unroll
        for (int G = 0; G < G16; ++G) {
#pragma unroll
            for (int r = 0; r < 4; ++r) rec[m.w_off[0] + (16 * G + 4 * q16 + r) * C + i16] = dW1t[G][r];
            float s1 = db1[G] + __shfl_xor(db1[G], 16, 64);
            s1 += __shfl_xor(s1, 32, 64);
            if (lane < 16) rec[m.b_off[0] + 16 * G + i16] = s1;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float s = H == 32 ? dWo[r] + __shfl_xor(dWo[r], 32, 64) : dWo[r];
        if (lane < H) rec[m.w_off[NH] + r * H + lane] = s;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float s = wave_sum(grp == 0 ? dbo[i] : 0.0f);
        if (lane == 0) rec[m.b_off[NH] + i] = s;
    }
}

template <int KIND, int C, int H, int NH, bool CC, int GT = LP_F32>
hipError_t launch_bwd_tile(const GridDev& g, const MlpDev& m, const RaysDev& rays, const BwdIo& io, int n_cu,
                           hipStream_t stream)
{
    using L = TileLds<C, H, NH>;
    auto kernel = bwd_tile_kernel<KIND, C, H, NH, CC, GT>;
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, L::kTotal);
    if (e != hipSuccess) return e;
    const int blocks = (n_cu + 7) / 8 * 8;
    // Tiles or single rays: the longest wave's number of steps decides.  A tile's step is cheaper to scatter, but a
    // launch of few rays spreads over more waves ray by ray.  Neighbouring rays, backward time in single rays over that
    // in tiles, for 16- and 32-channel voxel grids and triplanes and a hash table at 64 and 256 samples:
    // 1.03 .. 2.6 where a wave's steps are as many, 0.81 .. 1.65 at 1.33 times as many in tiles (16-channel voxels and the
    // hash table at 256 samples lose, 32 channels at 64 samples gain most), 0.68 .. 1.4 at 1.6 times.  The line stands
    // where no structure loses.  Patches against tiles alike.
    const long long n_tiles = (rays.M + kTileRays - 1) / kTileRays, n_patches = (rays.M + kPatchRays - 1) / kPatchRays;
    auto steps = [&](long long items, long long step) { return wave_steps<long long>(items, blocks, rays.S, step); };
    const bool tiles = 20 * steps(n_tiles, kTileSamples) <= 21 * steps(rays.M, 32);
    const bool patches = tiles && 20 * steps(n_patches, kPatchSamples) <= 21 * steps(n_tiles, kTileSamples) && rays.M < (1LL << 31);
    const TileSchedule sc = tile_schedule<long long>(patches ? Items::kPatches : tiles ? Items::kTiles : Items::kRays, tiles ? n_tiles : rays.M, blocks);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kTileWaves * 64), L::kTotal, stream, g, m, rays, io, sc);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_params_kernel, dim3((m.param_total + 63) / 64), dim3(kReduceThreads), 0, stream, m, io, blocks);
    return hipGetLastError();
}

template <int KIND>
hipError_t dispatch_bwd_tile(const GridDev& g, const MlpDev& m, const RaysDev& rays, const BwdIo& io, int n_cu,
                             hipStream_t stream)
{
    const int C = m.dims[0], H = m.dims[1], NH = m.n_layers - 1;
    if (g.C != C) return hipErrorInvalidValue;
    // grids stored in bf16 / fp16 take the contraction as a run-time branch (no second set of instantiations)
#define LP_CASE(c, h, nh)                                                                                       \
    if (C == c && H == h && NH == nh) {                                                                         \
        if (g.dtype == LP_BF16) return launch_bwd_tile<KIND, c, h, nh, false, LP_BF16>(g, m, rays, io, n_cu, stream); \
        if (g.dtype == LP_F16) return launch_bwd_tile<KIND, c, h, nh, false, LP_F16>(g, m, rays, io, n_cu, stream);   \
        return g.contract > 0.0 ? launch_bwd_tile<KIND, c, h, nh, true>(g, m, rays, io, n_cu, stream)           \
                                : launch_bwd_tile<KIND, c, h, nh, false>(g, m, rays, io, n_cu, stream);         \
    }
    LP_CASE(16, 32, 1) LP_CASE(16, 64, 1) LP_CASE(32, 32, 1) LP_CASE(32, 64, 1)
    LP_CASE(16, 32, 2) LP_CASE(16, 64, 2) LP_CASE(32, 32, 2) LP_CASE(32, 64, 2)
#undef LP_CASE
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace lp
