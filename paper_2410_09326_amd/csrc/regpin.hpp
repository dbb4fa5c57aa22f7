// Keeps a register tile's amplitudes in one block of vector registers.
//
// The tile kernel's operation loop is a switch over some 300 unrolled bodies that
// all read and write the whole tile.  Left to itself the register allocator
// places the amplitudes one by one, differently in different bodies, and
// joins the bodies with 100 and more register moves per operation.  An empty
// statement at the end of each body that takes the tile as 32-register tuples
// makes the tuple the unit of allocation.
#pragma once
#include <hip/hip_runtime.h>

namespace qops {

template <typename T, int N>
struct Tuple {
    using V = T __attribute__((ext_vector_type(N)));
};

// Amplitudes per tuple: 32 registers at most.
template <int N>
__device__ __forceinline__ void pin_tile(float2 (&a)[N])
{
    constexpr int M = N < 16 ? N : 16;
#pragma unroll
    for (int h = 0; h < N / M; ++h) {
        typename Tuple<float, 2 * M>::V v;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            v[2 * j] = a[M * h + j].x;
            v[2 * j + 1] = a[M * h + j].y;
        }
        asm volatile("" : "+v"(v));
#pragma unroll
        for (int j = 0; j < M; ++j) {
            a[M * h + j].x = v[2 * j];
            a[M * h + j].y = v[2 * j + 1];
        }
    }
}

template <int N>
__device__ __forceinline__ void pin_tile(double2 (&a)[N])
{
    constexpr int M = N < 8 ? N : 8;
#pragma unroll
    for (int h = 0; h < N / M; ++h) {
        typename Tuple<double, 2 * M>::V v;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            v[2 * j] = a[M * h + j].x;
            v[2 * j + 1] = a[M * h + j].y;
        }
        asm volatile("" : "+v"(v));
#pragma unroll
        for (int j = 0; j < M; ++j) {
            a[M * h + j].x = v[2 * j];
            a[M * h + j].y = v[2 * j + 1];
        }
    }
}

}  // namespace qops
