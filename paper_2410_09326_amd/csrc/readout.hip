// Readout of |psi_x|^2 in FP64 (paper Sec. II-B, IV-E): marginal
// distributions, <Z_q> and the norm, and two-qubit correlators <Z_a Z_b> for
// lists of pairs (what a diagonal cost Hamiltonian such as weighted Max-Cut's
// is assembled from).  Every kernel reads the state once, 16 bytes per thread
// and access and eight accesses ahead of their use, and sums in a fixed order,
// so results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"

namespace qops {
namespace {

constexpr int kThreads = 256;

// One 16-byte access of a state: two complex64 amplitudes (physical bit 0
// apart) or one complex128 amplitude.  A row is what a work-group reads with
// one access per thread: 2^kRowBits consecutive amplitudes.
// The state may start at any amplitude of a larger buffer, so the type claims
// no more than the amplitude's own alignment (the hardware takes 16-byte
// accesses at any multiple of four).
template <typename T>
struct Row;
using Amp2 = float __attribute__((ext_vector_type(4), aligned(8)));
template <>
struct Row<float> {
    using V = Amp2;
    static constexpr int kRowBits = 9;
};
template <>
struct Row<double> {
    using V = double2;
    static constexpr int kRowBits = 8;
};

// |amplitude|^2 added to acc.
__device__ __forceinline__ double add_prob(double re, double im, double acc)
{
    return __builtin_fma(im, im, __builtin_fma(re, re, acc));
}

// Bits of v, lowest first, placed at the set positions of mask.
__device__ __forceinline__ uint64_t deposit64(uint64_t v, uint64_t mask)
{
    uint64_t r = 0;
    while (mask) {
        const uint64_t low = mask & (0ull - mask);
        if (v & 1u) r |= low;
        v >>= 1;
        mask &= mask - 1u;
    }
    return r;
}

// Sum over the 64 lanes (butterfly, every lane gets it).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int w = 1; w < 64; w <<= 1) v += __shfl_xor(v, w, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Marginal probabilities
// ---------------------------------------------------------------------------

// out[y] = sum of p over the physical bits that are not marginal.  The high
// bits (those above a row) split into marginal ones, which number the
// work-groups, and free ones, which a work-group walks; `slice_mask` holds the
// free bits that are split over work-groups too where the marginal ones give
// too few of them, and their partial sums are added by probs_slices_kernel.
// A thread keeps one sum per amplitude of its access, so the state streams
// through registers; the row's own free bits are folded once at the end.
// HBM read bound: 8 of 28 bits of a complex64 state take 0.37 ms, 5.8 TB/s
// (before: 7.9-17 ms, a few threads adding up 4096 LDS values serially), 15 of
// 25 bits of a complex128 state 0.11 ms (before: 1.05 ms, one strided chain per
// output).
struct ProbsArgs {
    uint64_t it_mask;        // free high bits a work-group walks
    uint64_t slice_mask;     // free high bits that number slices
    uint64_t marg_mask;      // marginal high bits
    int it_bits, slice_bits, m, n;
    uint32_t low_free;       // free bits of the row
    int8_t low_out[9];       // output bit of row bit b, or -1
    int8_t high_out[QOPS_MAX_QUBITS_DEV];   // output bit of the i-th marginal high bit
    int n_high;
};

template <typename T>
__global__ void __launch_bounds__(kThreads)
probs_kernel(const typename Row<T>::V* __restrict__ st, ProbsArgs a, double* __restrict__ out)
{
    constexpr int RB = Row<T>::kRowBits, PER = RB - 8 + 1;   // amplitudes per access
    __shared__ double tab[1 << RB];
    const int t = threadIdx.x;
    const uint32_t block = blockIdx.y * gridDim.x + blockIdx.x;
    const uint64_t slice = block & ((1u << a.slice_bits) - 1u);
    const uint64_t high = block >> a.slice_bits;
    const uint64_t base = deposit64(slice, a.slice_mask) | deposit64(high, a.marg_mask);
    const bool in = a.n >= RB || (t * PER) < (1 << a.n);     // smaller states fill part of a row
    double s0 = 0.0, s1 = 0.0;
    auto p0 = [](const typename Row<T>::V v) { return add_prob((double)v.x, (double)v.y, 0.0); };
    auto p1 = [](const typename Row<T>::V v) {
        if constexpr (PER == 2) return add_prob((double)v.z, (double)v.w, 0.0);
        else return 0.0;
    };
    // eight rows are added as a tree before they join the running sum: an
    // eighth of the roundings of a plain chain
    auto tree = [](const double (&q)[8]) { return ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7])); };
    if (in) {
        const typename Row<T>::V* __restrict__ src = st + (base >> (PER - 1)) + t;
        if (a.it_bits >= 3) {
            uint64_t o[8];
            const uint64_t m0 = a.it_mask & (0ull - a.it_mask), r1 = a.it_mask ^ m0, m1 = r1 & (0ull - r1),
                           r2 = r1 ^ m1, m2 = r2 & (0ull - r2), rest = r2 ^ m2;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                o[k] = ((k & 1 ? m0 : 0) | (k & 2 ? m1 : 0) | (k & 4 ? m2 : 0)) >> (PER - 1);
            uint64_t x = 0;
            for (uint64_t i = 0; i < (1ull << (a.it_bits - 3)); ++i) {
                typename Row<T>::V v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = src[(x >> (PER - 1)) + o[k]];
                double q[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) q[k] = p0(v[k]);
                s0 += tree(q);
                if constexpr (PER == 2) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) q[k] = p1(v[k]);
                    s1 += tree(q);
                }
                x = ((x | ~rest) + 1) & rest;
            }
        } else {
            uint64_t x = 0;
            for (uint64_t i = 0; i < (1ull << a.it_bits); ++i) {
                const typename Row<T>::V v = src[x >> (PER - 1)];
                s0 += p0(v);
                s1 += p1(v);
                x = ((x | ~a.it_mask) + 1) & a.it_mask;
            }
        }
    }
    tab[t * PER] = s0;
    if constexpr (PER == 2) tab[t * PER + 1] = s1;
    __syncthreads();
    for (int b = RB - 1; b >= 0; --b) {
        if (!((a.low_free >> b) & 1u)) continue;
        for (int l = t; l < (1 << RB); l += kThreads)
            if (!((l >> b) & 1)) tab[l] += tab[l | (1 << b)];
        __syncthreads();
    }
    uint32_t yh = 0;
    for (int i = 0; i < a.n_high; ++i) yh |= (uint32_t)((high >> i) & 1u) << a.high_out[i];
    for (int l = t; l < (1 << RB); l += kThreads) {
        if ((uint32_t)l & a.low_free) continue;
        uint32_t y = yh;
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if (a.low_out[b] >= 0) y |= (uint32_t)((l >> b) & 1) << a.low_out[b];
        out[((uint64_t)y << a.slice_bits) + slice] = tab[l];
    }
}

// out[y] = sum over slices of part[y 2^slice_bits + slice]; one wave per y.
__global__ void __launch_bounds__(kThreads)
probs_slices_kernel(const double* __restrict__ part, int slice_bits, uint32_t ny, double* __restrict__ out)
{
    const uint32_t y = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (y >= ny) return;
    const double* __restrict__ p = part + ((uint64_t)y << slice_bits);
    double v = 0.0;
    for (uint32_t i = threadIdx.x & 63; i < (1u << slice_bits); i += 64) v += p[i];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) out[y] = v;
}

// All bits marginal: a permutation of |psi|^2, no sum.
template <typename T, typename V>
__global__ void __launch_bounds__(kThreads) probs_direct_kernel(const V* __restrict__ st, int n, PosArr pa,
                                                                double* __restrict__ out)
{
    const uint64_t N = 1ull << n;
    for (uint64_t x = blockIdx.x * (uint64_t)kThreads + threadIdx.x; x < N; x += (uint64_t)gridDim.x * kThreads) {
        uint64_t y = 0;
        for (int j = 0; j < n; ++j) y |= ((x >> pa.p[j]) & 1ull) << j;
        const V v = st[x];
        const double re = (double)v.x, im = (double)v.y;
        out[y] = re * re + im * im;
    }
}

template <typename T>
void probs_geometry(int n, int m, const int* pos, ProbsArgs& a)
{
    constexpr int RB = Row<T>::kRowBits;
    a = ProbsArgs{};
    a.n = n;
    a.m = m;
    int out_of[QOPS_MAX_QUBITS_DEV];
    for (int b = 0; b < QOPS_MAX_QUBITS_DEV; ++b) out_of[b] = -1;
    for (int j = 0; j < m; ++j) out_of[pos[j]] = j;
    for (int b = 0; b < RB; ++b) {
        a.low_out[b] = (int8_t)(b < n ? out_of[b] : -1);
        if (a.low_out[b] < 0) a.low_free |= 1u << b;
    }
    uint64_t free_mask = 0;
    int nfree = 0;
    for (int b = RB; b < n; ++b) {
        if (out_of[b] >= 0) {
            a.marg_mask |= 1ull << b;
            a.high_out[a.n_high++] = (int8_t)out_of[b];
        } else {
            free_mask |= 1ull << b;
            ++nfree;
        }
    }
    // 2^11 work-groups fill the chip (8 per CU) and still leave each enough
    // rows to hide its start and its folding behind; slices come from the
    // highest free bits and keep at least eight rows in each
    a.slice_bits = std::max(0, std::min(11 - a.n_high, nfree - 3));
    a.it_bits = nfree - a.slice_bits;
    int left = a.it_bits;
    for (int b = RB; b < n; ++b) {
        if (!((free_mask >> b) & 1ull)) continue;
        if (left > 0) {
            a.it_mask |= 1ull << b;
            --left;
        } else {
            a.slice_mask |= 1ull << b;
        }
    }
}

void probs_geometry(int prec, int n, int m, const int* pos, ProbsArgs& a)
{
    if (prec == 0) probs_geometry<float>(n, m, pos, a);
    else probs_geometry<double>(n, m, pos, a);
}

// ---------------------------------------------------------------------------
// <Z_q> and the norm
// ---------------------------------------------------------------------------

// Block b of B sums the chunk [b 2^s, (b+1) 2^s): part[b] = sum p,
// part[(1 + q) B + b] = sum p * bit_q(x).  Rows are taken in groups of
// eight, whose three bits a small addition tree separates; the bits above
// (OB of them at most) are uniform per group, so one conditional addition of
// the group's sum each.  HBM read bound: 30 qubits complex64 1.39 ms, 6.2 TB/s (before:
// 1.95 ms with one 8-byte load in flight per thread, an addition per amplitude
// and loop bit, and nine barriers per reduced value).
template <typename T, int OB>
__global__ void __launch_bounds__(kThreads)
zsum_part_kernel(const typename Row<T>::V* __restrict__ st, int n, int s, double* __restrict__ part)
{
    constexpr int RB = Row<T>::kRowBits, PER = RB - 8 + 1;
    constexpr int NV = RB + 3 + OB + 1;     // values a block reduces: sum p and one per bit below s
    __shared__ double sh[4][NV];
    const uint64_t base = (uint64_t)blockIdx.x << s;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int rbits = s > RB ? s - RB : 0;  // row number bits
    const int gbits = rbits > 3 ? rbits - 3 : 0;
    const int rows = rbits < 3 ? 1 << rbits : 8;
    const bool in = s >= RB || (t * PER) < (1 << s);
    double tot = 0.0, b0 = 0.0, l0 = 0.0, l1 = 0.0, l2 = 0.0, ob[OB];
#pragma unroll
    for (int k = 0; k < OB; ++k) ob[k] = 0.0;
    if (in) {
        const typename Row<T>::V* __restrict__ src = st + (base >> (PER - 1)) + t;
        for (uint32_t g = 0; g < (1u << gbits); ++g) {
            typename Row<T>::V v[8];
            const typename Row<T>::V* __restrict__ row = src + (size_t)g * 8 * kThreads;
            if (rows == 8) {
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = row[k * kThreads];
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    v[k] = typename Row<T>::V{};
                    if (k < rows) v[k] = row[k * kThreads];
                }
            }
            double q[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if constexpr (PER == 2) {
                    const double hi = add_prob((double)v[k].z, (double)v[k].w, 0.0);
                    b0 += hi;
                    q[k] = add_prob((double)v[k].x, (double)v[k].y, hi);
                } else {
                    q[k] = add_prob(v[k].x, v[k].y, 0.0);
                }
            }
            const double a0 = q[0] + q[1], a1 = q[2] + q[3], a2 = q[4] + q[5], a3 = q[6] + q[7];
            const double c1 = a2 + a3, sum = (a0 + a1) + c1;
            l0 += (q[1] + q[3]) + (q[5] + q[7]);
            l1 += a1 + a3;
            l2 += c1;
            tot += sum;
#pragma unroll
            for (int k = 0; k < OB; ++k)
                if ((g >> k) & 1u) ob[k] += sum;
        }
    }
    // value i of the block: 0 = sum p, 1 + b = sum p bit_b
    auto put = [&](int i, double v) {
        v = wave_sum(v);
        if (lane == 0) sh[wave][i] = v;
    };
    put(0, tot);
    if constexpr (PER == 2) put(1, b0);
#pragma unroll
    for (int b = 0; b < 6; ++b) put(PER + b, (lane >> b) & 1 ? tot : 0.0);
    put(PER + 6, wave & 1 ? tot : 0.0);
    put(PER + 7, wave & 2 ? tot : 0.0);
    put(RB + 1, l0);
    put(RB + 2, l1);
    put(RB + 3, l2);
#pragma unroll
    for (int k = 0; k < OB; ++k)
        if (k < gbits) put(RB + 4 + k, ob[k]);
    __syncthreads();
    if (t <= n) {
        const int i = t <= s ? t : 0;       // bits above the chunk: all or nothing
        double v = ((sh[0][i] + sh[1][i]) + sh[2][i]) + sh[3][i];
        if (t > s && !((base >> (t - 1)) & 1ull)) v = 0.0;
        part[(uint64_t)t * gridDim.x + blockIdx.x] = v;
    }
}

// One block per output quantity: sums part[qi*nparts + b] over blocks b.
__global__ void __launch_bounds__(kThreads) zsum_final_kernel(const double* __restrict__ part, int nparts,
                                                              double* __restrict__ out)
{
    __shared__ double sh[4];
    const int qi = blockIdx.x;
    double v = 0.0;
    for (int b = threadIdx.x; b < nparts; b += kThreads) v += part[(uint64_t)qi * nparts + b];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) out[qi] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// out[q] = sums[0] - 2 sums[1 + l2p[q]]: <Z_q> of logical qubit q.
__global__ void z_logical_kernel(const double* __restrict__ sums, int n, ZLayout lay, double* __restrict__ out)
{
    const int q = threadIdx.x;
    if (q < n) out[q] = sums[0] - 2.0 * sums[1 + lay.l2p[q]];
}

int zsum_chunk_bits(int n) { return n < 16 ? n : 16; }

// Chunks of 2^s amplitudes with s = max(zsum_chunk_bits(n), n - 11): at
// most 2^11 partial records whatever n is (up to 23 chunk bits at n = 34);
// for n <= 27 the chunks, and so the summation order, equal launch_zsum's.
int zsum_bounded_chunk_bits(int n) { return std::max(zsum_chunk_bits(n), n - 11); }

template <typename T>
void launch_zsum_part(const void* state, int n, int s, double* part, hipStream_t st)
{
    using V = typename Row<T>::V;
    const unsigned nb = 1u << (n - s);
    if (s <= 16)
        hipLaunchKernelGGL((zsum_part_kernel<T, 5>), dim3(nb), dim3(kThreads), 0, st,
                           reinterpret_cast<const V*>(state), n, s, part);
    else
        hipLaunchKernelGGL((zsum_part_kernel<T, 12>), dim3(nb), dim3(kThreads), 0, st,
                           reinterpret_cast<const V*>(state), n, s, part);
}

hipError_t launch_zsum_s(int prec, const void* state, int n, int s, double* part, double* out, hipStream_t st)
{
    if (prec == 0) launch_zsum_part<float>(state, n, s, part, st);
    else launch_zsum_part<double>(state, n, s, part, st);
    hipLaunchKernelGGL(zsum_final_kernel, dim3(n + 1), dim3(kThreads), 0, st, part, (int)(1u << (n - s)), out);
    return hipGetLastError();
}

}  // namespace

size_t zsum_scratch_doubles(int n)
{
    const int s = zsum_chunk_bits(n);
    return (size_t(1) << (n - s)) * (n + 1);
}

hipError_t launch_zsum(int prec, const void* state, int n, double* scratch, double* out, hipStream_t st)
{
    return launch_zsum_s(prec, state, n, zsum_chunk_bits(n), scratch, out, st);
}

size_t zsum_bounded_scratch_doubles(int n)
{
    return (size_t(1) << (n - zsum_bounded_chunk_bits(n))) * (n + 1) + (n + 1);
}

hipError_t launch_expect_z_bounded(int prec, const void* state, int n, const int32_t* l2p, double* scratch,
                                   double* out, hipStream_t st)
{
    if (n < 1 || n > QOPS_MAX_QUBITS_DEV) return hipErrorInvalidValue;
    const int s = zsum_bounded_chunk_bits(n);
    double* part = scratch;
    double* sums = scratch + (size_t(1) << (n - s)) * (n + 1);
    hipError_t e = launch_zsum_s(prec, state, n, s, part, sums, st);
    if (e != hipSuccess) return e;
    ZLayout lay;
    for (int q = 0; q < QOPS_MAX_QUBITS_DEV; ++q) lay.l2p[q] = q < n ? l2p[q] : 0;
    hipLaunchKernelGGL(z_logical_kernel, dim3(1), dim3(64), 0, st, sums, n, lay, out);
    return hipGetLastError();
}

size_t probs_scratch_doubles(int prec, int n, int m, const int* pos)
{
    if (m == n) return 0;
    ProbsArgs a;
    probs_geometry(prec, n, m, pos, a);
    return a.slice_bits > 0 ? size_t(1) << (m + a.slice_bits) : 0;
}

hipError_t launch_probs(int prec, const void* state, int n, int m, const int* pos, double* scratch, double* out,
                        hipStream_t st)
{
    if (m == n) {
        PosArr pa;
        for (int j = 0; j < QOPS_MAX_QUBITS_DEV; ++j) pa.p[j] = j < m ? pos[j] : 0;
        const unsigned grid = (unsigned)std::min<uint64_t>(((1ull << n) + kThreads - 1) / kThreads, 256ull * 64);
        if (prec == 0)
            hipLaunchKernelGGL((probs_direct_kernel<float, float2>), dim3(grid), dim3(kThreads), 0, st,
                               reinterpret_cast<const float2*>(state), n, pa, out);
        else
            hipLaunchKernelGGL((probs_direct_kernel<double, double2>), dim3(grid), dim3(kThreads), 0, st,
                               reinterpret_cast<const double2*>(state), n, pa, out);
        return hipGetLastError();
    }
    ProbsArgs a;
    probs_geometry(prec, n, m, pos, a);
    // one dimension of a dispatch holds fewer than 2^32 work-items, which 24
    // marginal high bits exceed: the numbers above 2^20 go to the second one
    const int bits = a.n_high + a.slice_bits, xbits = std::min(bits, 20);
    const dim3 grid(1u << xbits, 1u << (bits - xbits));
    double* dst = a.slice_bits > 0 ? scratch : out;
    if (prec == 0)
        hipLaunchKernelGGL(probs_kernel<float>, grid, dim3(kThreads), 0, st,
                           reinterpret_cast<const Amp2*>(state), a, dst);
    else
        hipLaunchKernelGGL(probs_kernel<double>, grid, dim3(kThreads), 0, st,
                           reinterpret_cast<const double2*>(state), a, dst);
    if (a.slice_bits > 0) {
        const uint32_t ny = 1u << m;
        hipLaunchKernelGGL(probs_slices_kernel, dim3((ny + 3) / 4), dim3(kThreads), 0, st, scratch, a.slice_bits, ny,
                           out);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// <Z_a Z_b>
// ---------------------------------------------------------------------------

namespace {

constexpr int kZZPairs = 64;     // pairs per read of the state

// A thread of zz_part_kernel sums over eight local bits of a 2^16-amplitude
// chunk: the three row bits of a group of eight rows, bit 0 (complex64) and
// the row number's higher bits.  A pair's sign splits into the part on the
// local bits -- none, one bit or two: 37 patterns, each with its own running
// sum -- and the part on the other bits, which is one sign per thread and
// chunk.  So all pairs of a launch share one read and one set of 37 sums
// (about 6 additions per amplitude), and each pair adds one signed reduction
// per chunk.  42 pairs at 28 qubits complex64: 0.45 ms, 4.7 TB/s (before: 3.35 ms, one
// read and 64-bit shifts per amplitude and pair for every eight pairs).
constexpr int kLocal = 8;
constexpr int kPatterns = 1 + kLocal + kLocal * (kLocal - 1) / 2;

// Pattern numbers: 0 = none, 1 + i = local bit i, 9 + ... = bits i < j.
__host__ __device__ constexpr int pattern1(int i) { return 1 + i; }
__host__ __device__ constexpr int pattern2(int i, int j) { return 1 + kLocal + i * (2 * kLocal - i - 1) / 2 + (j - i - 1); }

struct PairList {
    uint64_t far[kZZPairs];             // physical bits outside the local ones
    uint8_t slot[kZZPairs];             // result slot of the pair
    uint8_t first[kPatterns + 1];       // pairs of pattern k: [first[k], first[k + 1])
    int32_t count;
};

// Local bit order: c64: bit 0, row bits 9..11, then 12..15; c128: row bits
// 8..10, then 11..15.
template <typename T>
__host__ __device__ constexpr int local_bit(int i)
{
    return sizeof(T) == 4 ? (i == 0 ? 0 : 8 + i) : 8 + i;
}

template <typename T>
__global__ void __launch_bounds__(kThreads)
zz_part_kernel(const typename Row<T>::V* __restrict__ st, int n, uint32_t nchunks, PairList pl,
               double* __restrict__ part)
{
    constexpr int RB = Row<T>::kRowBits, PER = RB - 8 + 1;
    constexpr int R0 = PER - 1;                 // local index of the first row bit
    constexpr int O0 = R0 + 3, NO = kLocal - O0;   // higher row-number bits
    __shared__ double sh[4][kZZPairs];
    __shared__ double acc[kZZPairs];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int s = n < 16 ? n : 16;
    const int rbits = s > RB ? s - RB : 0;
    const int gbits = rbits > 3 ? rbits - 3 : 0;
    const int rows = rbits < 3 ? 1 << rbits : 8;
    const bool in = s >= RB || (t * PER) < (1 << s);
    if (t < kZZPairs) acc[t] = 0.0;
    for (uint32_t chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x) {
        const uint64_t base = (uint64_t)chunk << s;
        double S[kPatterns];
#pragma unroll
        for (int k = 0; k < kPatterns; ++k) S[k] = 0.0;
        const typename Row<T>::V* __restrict__ src = st + (base >> (PER - 1)) + t;
        for (uint32_t g = 0; g < (1u << gbits); ++g) {
            const typename Row<T>::V* __restrict__ row = src + (size_t)g * 8 * kThreads;
            typename Row<T>::V v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                v[k] = typename Row<T>::V{};
                if (in && k < rows) v[k] = row[k * kThreads];
            }
            double q[8], d[8];                  // sum and (complex64) difference over bit 0
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if constexpr (PER == 2) {
                    const double lo = add_prob((double)v[k].x, (double)v[k].y, 0.0);
                    const double hi = add_prob((double)v[k].z, (double)v[k].w, 0.0);
                    q[k] = lo + hi;
                    d[k] = lo - hi;
                } else {
                    q[k] = add_prob(v[k].x, v[k].y, 0.0);
                    d[k] = 0.0;
                }
            }
            // Walsh-Hadamard transform over the three row bits
            auto wht = [](double (&w)[8]) {
#pragma unroll
                for (int h = 1; h < 8; h <<= 1)
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (!(k & h)) {
                            const double x = w[k], y = w[k | h];
                            w[k] = x + y;
                            w[k | h] = x - y;
                        }
            };
            wht(q);
            if constexpr (PER == 2) wht(d);
            S[0] += q[0];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                S[pattern1(R0 + i)] += q[1 << i];
#pragma unroll
                for (int j = i + 1; j < 3; ++j) S[pattern2(R0 + i, R0 + j)] += q[(1 << i) | (1 << j)];
            }
            if constexpr (PER == 2) {
                S[pattern1(0)] += d[0];
#pragma unroll
                for (int i = 0; i < 3; ++i) S[pattern2(0, R0 + i)] += d[1 << i];
            }
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                const double so = (g >> o) & 1u ? -1.0 : 1.0;
                S[pattern1(O0 + o)] = __builtin_fma(so, q[0], S[pattern1(O0 + o)]);
                if constexpr (PER == 2) S[pattern2(0, O0 + o)] = __builtin_fma(so, d[0], S[pattern2(0, O0 + o)]);
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    S[pattern2(R0 + i, O0 + o)] = __builtin_fma(so, q[1 << i], S[pattern2(R0 + i, O0 + o)]);
#pragma unroll
                for (int p = o + 1; p < NO; ++p) {
                    const double sp = ((g >> o) ^ (g >> p)) & 1u ? -1.0 : 1.0;
                    S[pattern2(O0 + o, O0 + p)] = __builtin_fma(sp, q[0], S[pattern2(O0 + o, O0 + p)]);
                }
            }
        }
        const uint64_t x = base | ((uint64_t)t << (PER - 1));
#pragma unroll
        for (int k = 0; k < kPatterns; ++k)
            for (int i = pl.first[k]; i < pl.first[k + 1]; ++i) {
                const double w = wave_sum(__popcll(x & pl.far[i]) & 1 ? -S[k] : S[k]);
                if (lane == 0) sh[wave][i] = w;
            }
        __syncthreads();
        if (t < pl.count) acc[t] += ((sh[0][t] + sh[1][t]) + sh[2][t]) + sh[3][t];
        __syncthreads();
    }
    if (t < pl.count) part[(size_t)pl.slot[t] * gridDim.x + blockIdx.x] = acc[t];
}

// out[c] = sum over blocks g of part[c nblocks + g], in a fixed order.
__global__ void __launch_bounds__(kThreads)
zz_final_kernel(const double* __restrict__ part, int nblocks, double* __restrict__ out)
{
    __shared__ double sh[4];
    const double* __restrict__ p = part + (size_t)blockIdx.x * nblocks;
    double v = 0.0;
    for (int g = threadIdx.x; g < nblocks; g += kThreads) v += p[g];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

unsigned zz_blocks(int n) { return n <= 16 ? 1u : (unsigned)std::min<uint64_t>(4096, 1ull << (n - 16)); }

template <typename T>
void zz_pattern(uint64_t mask, int& pattern, uint64_t& far)
{
    int bit[2], nb = 0;
    far = mask;
    for (int i = 0; i < kLocal; ++i)
        if (mask >> local_bit<T>(i) & 1ull) {
            bit[nb++] = i;
            far &= ~(1ull << local_bit<T>(i));
        }
    pattern = nb == 0 ? 0 : nb == 1 ? pattern1(bit[0]) : pattern2(bit[0], bit[1]);
}

}  // namespace

size_t zz_scratch_doubles(int n) { return (size_t)zz_blocks(n) * kZZPairs; }

hipError_t launch_expect_zz(int prec, const void* state, int n, const int32_t* pa, const int32_t* pb, int npairs,
                            double* part, double* d_out, hipStream_t s)
{
    const unsigned nb = zz_blocks(n);
    const uint32_t nchunks = n <= 16 ? 1u : 1u << (n - 16);
    for (int p0 = 0; p0 < npairs; p0 += kZZPairs) {
        PairList pl{};
        pl.count = std::min(kZZPairs, npairs - p0);
        int pattern[kZZPairs];
        uint64_t far[kZZPairs];
        for (int c = 0; c < pl.count; ++c) {
            const uint64_t mask = (1ull << pa[p0 + c]) ^ (1ull << pb[p0 + c]);   // a == b: no sign
            if (prec == 0) zz_pattern<float>(mask, pattern[c], far[c]);
            else zz_pattern<double>(mask, pattern[c], far[c]);
        }
        int at = 0;
        for (int k = 0; k < kPatterns; ++k) {
            pl.first[k] = (uint8_t)at;
            for (int c = 0; c < pl.count; ++c)
                if (pattern[c] == k) {
                    pl.far[at] = far[c];
                    pl.slot[at++] = (uint8_t)c;
                }
        }
        pl.first[kPatterns] = (uint8_t)at;
        if (prec == 0)
            hipLaunchKernelGGL(zz_part_kernel<float>, dim3(nb), dim3(kThreads), 0, s,
                               reinterpret_cast<const Amp2*>(state), n, nchunks, pl, part);
        else
            hipLaunchKernelGGL(zz_part_kernel<double>, dim3(nb), dim3(kThreads), 0, s,
                               reinterpret_cast<const double2*>(state), n, nchunks, pl, part);
        hipLaunchKernelGGL(zz_final_kernel, dim3((unsigned)pl.count), dim3(kThreads), 0, s, part, (int)nb, d_out + p0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qops
