// Keeps a register tile's amplitudes in one block of vector registers.
//
// The tile kernel's operation loop is a switch over ~100 unrolled bodies that
// all read and write the whole tile.  Left to itself the register allocator
// places the amplitudes one by one, differently in different bodies, and
// joins the bodies with 100 and more register moves per operation.  An empty
// statement at the end of each body that takes the tile as 32-register tuples
// makes the tuple the unit of allocation.
#pragma once
#include <hip/hip_runtime.h>

namespace qops {

using F32x32 = float __attribute__((ext_vector_type(32)));
using F64x16 = double __attribute__((ext_vector_type(16)));

template <int N>
__device__ __forceinline__ void pin_tile(float2 (&a)[N])
{
#pragma unroll
    for (int h = 0; h < N / 16; ++h) {
        F32x32 v;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            v[2 * j] = a[16 * h + j].x;
            v[2 * j + 1] = a[16 * h + j].y;
        }
        asm volatile("" : "+v"(v));
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            a[16 * h + j].x = v[2 * j];
            a[16 * h + j].y = v[2 * j + 1];
        }
    }
}

template <int N>
__device__ __forceinline__ void pin_tile(double2 (&a)[N])
{
#pragma unroll
    for (int h = 0; h < N / 8; ++h) {
        F64x16 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            v[2 * j] = a[8 * h + j].x;
            v[2 * j + 1] = a[8 * h + j].y;
        }
        asm volatile("" : "+v"(v));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            a[8 * h + j].x = v[2 * j];
            a[8 * h + j].y = v[2 * j + 1];
        }
    }
}

}  // namespace qops
