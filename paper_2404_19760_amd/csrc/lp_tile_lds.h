// LDS images of the tile kernels: bf16 matrices that are read both along their rows (as they were
// written) and along their columns (as the operand of a contraction over the rows), without a second
// copy and without transposing them on the matrix cores.
//
// A matrix of R rows and N columns (N = 16, 32 or 64) is kept as two images, the hi and the lo halves of
// the fp32 values, each R rows of N / 8 chunks of 16 bytes (8 bf16 values).  Row access moves whole
// chunks: a lane (i, g) of a 32-column matrix-core operand owns chunk 2s + g of row i in K-step s.  Column
// access uses the transposing LDS read of gfx950 (16 lanes point at the 8-byte quarters of a 4 x 16 block and
// receive its 16 columns, four rows each): two of them give the 8 elements of an operand over 16 rows.
//
// Chunks are stored at position `chunk ^ swizzle(row)` of their row, so that both kinds of access touch
// every bank once: row access takes one chunk of 16 consecutive rows, column access 32 (or 16) consecutive
// columns of four rows r, r + 1, r + 2, r + 3.
//
// Order of the columns inside a row:
//   hidden tensors  chunk 2s + g holds features 16 s + 4 g + {0..3} and 16 s + 8 + 4 g + {0..3}: the 8 values a
//                   lane of group g owns of a layer's output registers (k_hidden), packed as they are
//   inputs          natural order (k_input: lane group g owns the g-th half of the channels)
// Order of the rows in a column access: element e of lane group g in K-step s stands for row
// 16 s + 8 (e / 4) + 4 g + e % 4, the same for both operands of a contraction.
#pragma once
#include "lp_mfma.h"

namespace lp {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

// LDS by byte address: the kernels keep a few lane-dependent base addresses in registers and reach everything
// else from them with constant offsets and exclusive-ors.
typedef __attribute__((address_space(3))) char LdsByte;
template <class T>
__device__ __forceinline__ T lds_get(uint32_t at)
{
    typedef __attribute__((address_space(3))) const T LdsT;
    return *(LdsT*)(uintptr_t)(at);
}
template <class T>
__device__ __forceinline__ void lds_put(uint32_t at, T v)
{
    typedef __attribute__((address_space(3))) T LdsT;
    *(LdsT*)(uintptr_t)(at) = v;
}
__device__ __forceinline__ Frag lds_chunk(uint32_t at) { return __builtin_bit_cast(Frag, lds_get<u32x4>(at)); }
__device__ __forceinline__ void lds_put_chunk(uint32_t at, const Frag& f) { lds_put<u32x4>(at, __builtin_bit_cast(u32x4, f)); }

// four rows' values of one column per lane (see above); the address is this lane's 8-byte quarter
__device__ __forceinline__ s16x4 lds_tr(uint32_t at)
{
    typedef __attribute__((address_space(3))) s16x4 LdsS16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsS16x4*)(uintptr_t)(at));
}
__device__ __forceinline__ void lds_read_tr(uint32_t at, uint32_t& d0, uint32_t& d1)
{
    const u32x2 u = __builtin_bit_cast(u32x2, lds_tr(at));
    d0 = u[0];
    d1 = u[1];
}

// Keeps an address that never changes from being expanded, outside the step loop, into one register per
// access: to the compiler it is a new value here.
__device__ __forceinline__ void refresh(uint32_t& at) { asm volatile("" : "+v"(at)); }

template <int N, bool HIDDEN>
struct TileImage {
    static constexpr int kChunks = N / 8;
    static constexpr int kRow = N * 2;  // bytes
    static constexpr int bytes(int rows) { return rows * kRow; }   // of one image (hi or lo)

    __host__ __device__ static constexpr int swizzle(int row)
    {
        if (kChunks == 8) return ((row >> 1) & 1) * 4 + ((row >> 2) & 1) * 2 + ((row >> 3) & 1);
        if (kChunks == 4) return (row >> 2) & 3;
        return (row >> 3) & 1;
    }
    // Row access: byte offset of this lane group's chunk of row (lane & 31) in K-step 0; own_step(s) turns it
    // (exclusive or) into K-step s's. Rows of 32-row blocks share the swizzle: block b adds 32 b kRow.
    __device__ static __forceinline__ uint32_t own(int lane)
    {
        const int row = lane & 31, g = lane >> 5;
        return row * kRow + (((HIDDEN ? g : g * (N / 16)) ^ swizzle(row)) << 4);
    }
    static constexpr uint32_t own_step(int s) { return HIDDEN ? 32 * s : 16 * s; }
    // Column access, 32 columns per operand (lane & 31), 16 rows per K-step (+ 4 g, + 8 for the second half:
    // kHalf, exclusive or); N = 16: the 16 columns twice.  Column block nb: exclusive or 64 nb; K-step ks adds
    // 16 ks kRow.
    __device__ static __forceinline__ uint32_t col32(int lane)
    {
        const int q = lane >> 4, t = lane & 15;
        return at(4 * (q >> 1) + (t >> 2), N == 16 ? 0 : (q & 1), t);
    }
    // Column access, 16 columns per operand (lane & 15), 32 rows: column group G: exclusive or 32 G.
    __device__ static __forceinline__ uint32_t col16(int lane)
    {
        const int q = lane >> 4, t = lane & 15;
        return at(16 * (q >> 1) + 4 * (q & 1) + (t >> 2), 0, t);
    }
    static constexpr uint32_t kHalf = 8 * kRow | (swizzle(8) << 4);
    // Column access, one column per lane (N = 64; N = 32: the upper lanes take rows 16 .. 31), four rows: rows
    // 4 n ..: exclusive or rows4(n) for n < 4, then 16 kRow per four.
    __device__ static __forceinline__ uint32_t col64(int lane)
    {
        const int t = lane & 15;
        return at((N == 32 ? 16 * (lane >> 5) : 0) + (t >> 2), N == 32 ? (lane >> 4) & 1 : lane >> 4, t);
    }
    static constexpr uint32_t rows4(int n) { return 4 * n * kRow | (swizzle(4 * n) << 4); }

    // operand fragments from the addresses col32 / col16 (column block flipped in); `offset`: K-step and image, a
    // constant that the instruction adds
    __device__ static __forceinline__ Frag read(uint32_t at, int offset)
    {
        Frag f;
        lds_read_tr(at + offset, f.d[0], f.d[1]);
        lds_read_tr((at ^ kHalf) + offset, f.d[2], f.d[3]);
        return f;
    }

private:
    __device__ static __forceinline__ uint32_t at(int row, int G, int t)
    {
        const int c = t & 3;   // columns 16 G + 4 c ..
        const int chunk = 2 * G + (HIDDEN ? (c & 1) : (c >> 1)), half = HIDDEN ? (c >> 1) : (c & 1);
        return row * kRow + ((chunk ^ swizzle(row)) << 4) + half * 8;
    }
};

// Stages a weight matrix W [rows][ld] (its first N columns) as the two images at dst and dst + bytes(rows).
template <class Image, int N, bool HIDDEN>
__device__ __forceinline__ void stage_image(uint32_t dst, const float* __restrict__ W, int rows, int ld)
{
    constexpr int kChunks = Image::kChunks;
    for (int idx = threadIdx.x; idx < rows * kChunks; idx += blockDim.x) {
        const int row = idx / kChunks, chunk = idx % kChunks;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = HIDDEN ? 16 * (chunk >> 1) + 8 * (e / 4) + 4 * (chunk & 1) + (e % 4) : 8 * chunk + e;
            x[e] = W[(size_t)row * ld + c];
        }
        Frag hi, lo;
        split8(x, hi, lo);
        const uint32_t p = dst + row * Image::kRow + ((chunk ^ Image::swizzle(row)) << 4);
        lds_put_chunk(p, hi);
        lds_put_chunk(p + Image::bytes(rows), lo);
    }
}

}  // namespace lp
