// Alternating matrix products and vector work in one instruction stream.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace lp {

// Alternates N matrix products with U pieces of vector work that do not wait for them, in exactly this order
// (the pieces start after SKIP products). A 32 x 32 x 16 product occupies the matrix cores for 32 cycles, in
// which the same wave can issue eight vector instructions: measured on this chip, 24 products and 192
// multiply-adds take 1770 cycles one after the other and 1190 alternating (1330 and 1090 per wave with two waves
// on the SIMD).
//
// The compiler moves instructions without side effects across scheduling barriers, so each result is pinned in its
// place by an empty asm statement.
template <class T>
__device__ __forceinline__ void pin(T& v) { asm volatile("" : "+v"(v)); }

template <int I, int END, class F>
__device__ __forceinline__ void repeat(F& f)
{
    if constexpr (I < END) {
        f(std::integral_constant<int, I>());
        repeat<I + 1, END>(f);
    }
}
template <int N, int U, int SKIP, int I = 0, class P, class V>
__device__ __forceinline__ void weave(P& product, V& piece)
{
    if constexpr (I < N) {
        product(std::integral_constant<int, I>());
        constexpr int from = I <= SKIP ? 0 : U * (I - SKIP) / (N - SKIP), to = I < SKIP ? 0 : U * (I + 1 - SKIP) / (N - SKIP);
        repeat<from, to>(piece);
        __builtin_amdgcn_sched_barrier(0);
        weave<N, U, SKIP, I + 1>(product, piece);
    }
}

}  // namespace lp
