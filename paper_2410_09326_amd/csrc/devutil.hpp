// Device helpers shared by the kernel files: compile-time loops, complex
// arithmetic, LDS swizzle and index spreading.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "devprog.hpp"

namespace qops {


// Compile-time loop: calls f(std::integral_constant<int, I>) for I = 0..N-1,
// so that every register index is a constant and the state stays in VGPRs.
template <int I, int N, typename F>
__device__ __forceinline__ void sfor_impl(F& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        sfor_impl<I + 1, N>(f);
    }
}
template <int N, typename F>
__device__ __forceinline__ void sfor(F&& f)
{
    sfor_impl<0, N>(f);
}

template <typename T> struct CxT;
template <> struct CxT<float> { using V = float2; using A4 = float __attribute__((ext_vector_type(4))); };
template <> struct CxT<double> { using V = double2; using A4 = double __attribute__((ext_vector_type(4))); };

template <typename V>
__device__ __forceinline__ V cmul(V a, V b)
{
    V r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}

// m0*x0 + m1*x1 (complex)
template <typename V>
__device__ __forceinline__ V cdot2(V m0, V x0, V m1, V x1)
{
    V r;
    r.x = m0.x * x0.x - m0.y * x0.y + m1.x * x1.x - m1.y * x1.y;
    r.y = m0.x * x0.y + m0.y * x0.x + m1.x * x1.y + m1.y * x1.x;
    return r;
}

// Component-wise select by value (a conditional on two struct lvalues would
// select an address and pin the register array in scratch memory).
template <typename V>
__device__ __forceinline__ V csel(bool c, V a, V b)
{
    V r;
    r.x = c ? a.x : b.x;
    r.y = c ? a.y : b.y;
    return r;
}

template <typename T>
__device__ __forceinline__ typename CxT<T>::V ldc(const T* __restrict__ c, int i)
{
    typename CxT<T>::V v;
    v.x = c[2 * i];
    v.y = c[2 * i + 1];
    return v;
}

// Fused multiply-add in the state precision.
__device__ __forceinline__ float fmat(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmat(double a, double b, double c) { return __builtin_fma(a, b, c); }

// LDS slot of tile element e: the low five bits (32 amplitudes = one row of
// the 64 four-byte banks for complex64) are XORed with the next five, so
// that strided groups and matrix-core column sets spread over the banks.
// A bijection on [0, 2^L) for every L >= 5.
// GF(2)-linear: swz(a ^ b) = swz(a) ^ swz(b).
__host__ __device__ constexpr uint32_t swz(uint32_t e) { return e ^ ((e >> 5) & 31u); }

// Inserts a zero bit at every set position of `mask` (ascending) into g.
__device__ __forceinline__ uint32_t spread_mask(uint32_t g, uint32_t mask)
{
    while (mask) {
        const int p = __builtin_ctz(mask);
        mask &= mask - 1;
        const uint32_t low = g & ((1u << p) - 1u);
        g = ((g >> p) << (p + 1)) | low;
    }
    return g;
}

// Bits of g, lowest first, placed at the set positions of dmask (lowest first).
__device__ __forceinline__ uint32_t deposit_bits(uint32_t g, uint32_t dmask)
{
    uint32_t r = 0;
    while (dmask) {
        const uint32_t low = dmask & (0u - dmask);
        if (g & 1u) r |= low;
        g >>= 1;
        dmask &= dmask - 1u;
    }
    return r;
}

__device__ __forceinline__ uint64_t spread_mask64(uint64_t g, uint64_t mask)
{
    while (mask) {
        const int p = __builtin_ctzll(mask);
        mask &= mask - 1;
        const uint64_t low = g & ((1ull << p) - 1ull);
        g = ((g >> p) << (p + 1)) | low;
    }
    return g;
}

}  // namespace qops
