// Register tile pass: a wave holds 2^(6+R) amplitudes of the state in its
// registers (2^(6+R+W) in a work-group of 2^W waves), runs every operation of
// a pass on them and writes them back.  Also the batched form of the same
// body (pass p of many circuits in one launch).  The file is compiled once per
// variant (QOPS_RT_T, QOPS_RT_R, QOPS_RT_W given: the kernels and launches of
// one precision and register/wave split) and once without (the dispatch).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "devprog.hpp"
#include "devutil.hpp"
#include "kernels.hpp"
#include "regpin.hpp"
#include "regtile.hpp"

#ifdef QOPS_RT_T

namespace qops {

// ---------------------------------------------------------------------------
// Register-resident operations
// ---------------------------------------------------------------------------

// The tile stays in one register tuple only if no body needs an amplitude's
// old value after writing its new one (the allocator would otherwise keep two
// tuples and copy between them after every operation).  Bodies that update
// out of place exchange or copy explicitly; the others order their steps.
__device__ __forceinline__ void swap_reg(float& x, float& y) { asm("v_swap_b32 %0, %1" : "+v"(x), "+v"(y)); }
__device__ __forceinline__ void swap_reg(double& x, double& y)
{
    int2 a = __builtin_bit_cast(int2, x), b = __builtin_bit_cast(int2, y);
    asm("v_swap_b32 %0, %1" : "+v"(a.x), "+v"(b.x));
    asm("v_swap_b32 %0, %1" : "+v"(a.y), "+v"(b.y));
    x = __builtin_bit_cast(double, a);
    y = __builtin_bit_cast(double, b);
}
// Exchange where mask is all ones (bits only, so the values are untouched).
__device__ __forceinline__ void swap_masked(float& x, float& y, int mask)
{
    const int a = __float_as_int(x), b = __float_as_int(y), d = (a ^ b) & mask;
    x = __int_as_float(a ^ d);
    y = __int_as_float(b ^ d);
}
__device__ __forceinline__ void swap_masked(double& x, double& y, int mask)
{
    const long long a = __double_as_longlong(x), b = __double_as_longlong(y), d = (a ^ b) & (long long)mask;
    x = __longlong_as_double(a ^ d);
    y = __longlong_as_double(b ^ d);
}
__device__ __forceinline__ void put_reg(float2& d, const float2 v)
{
    asm("v_mov_b32 %0, %1" : "=v"(d.x) : "v"(v.x));
    asm("v_mov_b32 %0, %1" : "=v"(d.y) : "v"(v.y));
}
__device__ __forceinline__ void put_reg(double2& d, const double2 v)
{
    asm("v_mov_b64 %0, %1" : "=v"(d.x) : "v"(v.x));
    asm("v_mov_b64 %0, %1" : "=v"(d.y) : "v"(v.y));
}

// Steps that have to end in the amplitude's own registers, in an order in which
// no old value is needed after its register is overwritten.
#define QOPS_IN_PLACE(T, FMA, MOV)                                                                           \
    /* a = a b given t = a.y b.y, u = a.y b.x */                                                             \
    __device__ __forceinline__ void cmul_tail(T& ax, T& ay, T bx, T by, T t, T u)                            \
    {                                                                                                        \
        asm(FMA " %1, %0, %3, %5\n\t" FMA " %0, %0, %2, -%4" : "+v"(ax), "=&v"(ay) : "v"(bx), "v"(by), "v"(t), "v"(u)); \
    }                                                                                                        \
    /* a = t + i c a.y, u + c' a.y: ax = t - ci ay, ay = u + cr ay */                                         \
    __device__ __forceinline__ void ex_tail(T& ax, T& ay, T cr, T ci, T t, T u)                              \
    {                                                                                                        \
        asm(FMA " %0, -%2, %1, %4\n\t" FMA " %1, %3, %1, %5" : "=&v"(ax), "+v"(ay) : "v"(ci), "v"(cr), "v"(t), "v"(u)); \
    }                                                                                                        \
    /* x = p + c x */                                                                                        \
    __device__ __forceinline__ void ex_real(T& x, T c, T p) { asm(FMA " %0, %1, %0, %2" : "+v"(x) : "v"(c), "v"(p)); } \
    /* ax = p - ci ay, ay = u */                                                                             \
    __device__ __forceinline__ void ex_imag(T& ax, T& ay, T ci, T p, T u)                                    \
    {                                                                                                        \
        asm(FMA " %0, -%2, %1, %3\n\t" MOV " %1, %4" : "=&v"(ax), "+v"(ay) : "v"(ci), "v"(p), "v"(u));       \
    }
QOPS_IN_PLACE(float, "v_fma_f32", "v_mov_b32")
QOPS_IN_PLACE(double, "v_fma_f64", "v_mov_b64")
#undef QOPS_IN_PLACE

// a *= b (complex), in place.
template <typename V>
__device__ __forceinline__ void cmul_to(V& a, const V b)
{
    const auto t = a.y * b.y;
    const auto u = a.y * b.x;
    cmul_tail(a.x, a.y, b.x, b.y, t, u);
}

// Exact X on register bit B: exchange the two halves (no arithmetic).
// CTRL: 0 = none, 1 = controls outside the registers (`tok`, the per-lane
// result), 2 = any (and the slots whose bits `creg` equal `cval`, which is
// uniform per slot).
template <int B, int R, int CTRL, typename V>
__device__ __forceinline__ void xgate_reg_b(V (&a)[1 << R], uint32_t creg, uint32_t cval, bool tok)
{
    const int mask = tok ? -1 : 0;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int j1 = j | (1 << B);
            if (CTRL < 2 || ((uint32_t)j & creg) == cval) {
                if (CTRL) {
                    swap_masked(a[j].x, a[j1].x, mask);
                    swap_masked(a[j].y, a[j1].y, mask);
                } else {
                    swap_reg(a[j].x, a[j1].x);
                    swap_reg(a[j].y, a[j1].y);
                }
            }
        }
    });
    pin_tile(a);
}

// Full 2x2 on register bit B; CTRL as above.
template <int B, int R, int CTRL, typename V>
__device__ __forceinline__ void oneq_reg_b(V (&a)[1 << R], V m00, V m01, V m10, V m11, uint32_t creg, uint32_t cval, bool tok)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int j1 = j | (1 << B);
            if (CTRL < 2 || ((uint32_t)j & creg) == cval) {
                const V x0 = a[j], x1 = a[j1];
                const V y0 = cdot2(m00, x0, m01, x1);
                const V y1 = cdot2(m10, x0, m11, x1);
                if (CTRL) {
                    const V t = csel(tok, y0, x0), u = csel(tok, y1, x1);
                    put_reg(a[j], t);
                    put_reg(a[j1], u);
                } else {
                    put_reg(a[j], y0);
                    put_reg(a[j1], y1);
                }
            }
        }
    });
    pin_tile(a);
}

// Bodies whose register condition is known at compile time: slots whose bits
// in M equal VAL.
template <int R, uint32_t M, uint32_t VAL, typename T, typename V>
__device__ __forceinline__ void sign_slots(V (&a)[1 << R], T sgn)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (((uint32_t)j & M) == VAL) {
            a[j].x *= sgn;
            a[j].y *= sgn;
        }
    });
    pin_tile(a);
}

template <int R, uint32_t M, uint32_t VAL, typename V>
__device__ __forceinline__ void phase_slots(V (&a)[1 << R], const V ph)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (((uint32_t)j & M) == VAL) cmul_to(a[j], ph);
    });
    pin_tile(a);
}

// Slots times the table entry of their register bits MA, MB (0: none):
// p0, p1 (MA set), p2 (MB set), p3 (both).  Tables of at most two bits carry
// their entries in the record: fetched through the vector cache they cost an
// RZZ and a RY on register bits 0.62 us an operation at 20 qubits (complex64),
// now 0.34.
template <int R, uint32_t MA, uint32_t MB, typename V>
__device__ __forceinline__ void mul_slots(V (&a)[1 << R], const V p0, const V p1, const V p2, const V p3)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr uint32_t j = decltype(jc)::value;
        if constexpr ((j & MA) && (j & MB)) cmul_to(a[j], p3);
        else if constexpr ((j & MB) != 0u) cmul_to(a[j], p2);
        else if constexpr ((j & MA) != 0u) cmul_to(a[j], p1);
        else cmul_to(a[j], p0);
    });
    pin_tile(a);
}

// Diagonal table with one or two register bits MA, MB (0: none) at the table
// index bits named in `aux`.
template <typename T, int R, uint32_t MA, uint32_t MB, typename V>
__device__ __forceinline__ void diag_regs(V (&a)[1 << R], const T* __restrict__ tab, uint32_t ithr, int aux)
{
    const uint32_t ia = 1u << (aux >> 16 & 7), ib = MB ? 1u << (aux >> 19 & 7) : 0u;
    const V p0 = ldc(tab, (int)ithr), p1 = ldc(tab, (int)(ithr ^ ia));
    V p2 = p0, p3 = p1;
    if constexpr (MB != 0u) {
        p2 = ldc(tab, (int)(ithr ^ ib));
        p3 = ldc(tab, (int)(ithr ^ ia ^ ib));
    }
    mul_slots<R, MA, MB>(a, p0, p1, p2, p3);
}

template <int B, int R, uint32_t M, uint32_t VAL, typename V>
__device__ __forceinline__ void cx_slots(V (&a)[1 << R])
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B)) && ((uint32_t)j & M) == VAL) {
            swap_reg(a[j].x, a[j | (1 << B)].x);
            swap_reg(a[j].y, a[j | (1 << B)].y);
        }
    });
    pin_tile(a);
}

// Two-step (sheared) form of a 2x2 on register bit B: p += w q, then
// q += v p, with p the slots whose bit is FORM (0 or 1) and q the others.
// The 2x2 it stands for is diag(d0, d1) times this, possibly with the two
// slots exchanged; the planner carries the diagonal into the next operation
// on that bit and the exchange into later operations' slot conditions and
// indices (RegOpT::ctl and aux) and the store (PassHdr::flip).  Both steps update in place: 4 fused multiply-adds per
// amplitude (2 where w and v are real or imaginary) and no copies, against 8
// and two copies for the full product.  The kernel's bound is the vector
// ALU's issue rate, so that is its time: a 28-qubit QFT + 40 layers of U3 and
// CZ (complex64) went from 133.5 to 84.3 ms, of which about 36 ms by the
// arithmetic and 12 ms by keeping the tile in place (regpin.hpp).
// TY: 0 = complex, 1 = real, 2 = imaginary coefficients.
template <int TY, typename T, typename V>
__device__ __forceinline__ void axpy(V& p, T cr, T ci, const V q)
{
    if constexpr (TY != 2) {
        p.x = fmat(cr, q.x, p.x);
        p.y = fmat(cr, q.y, p.y);
    }
    if constexpr (TY != 1) {
        p.x = fmat(-ci, q.y, p.x);
        p.y = fmat(ci, q.x, p.y);
    }
}

template <int B, int R, int FORM, int TY, typename T, typename V>
__device__ __forceinline__ void shear_reg_b(V (&a)[1 << R], T wr, T wi, T vr, T vi)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int jp = FORM == 0 ? j : (j | (1 << B)), jq = j + (j | (1 << B)) - jp;
            axpy<TY>(a[jp], wr, wi, a[jq]);
            axpy<TY>(a[jq], vr, vi, a[jp]);
        }
    });
    pin_tile(a);
}

// Cross-lane exchange through ds_bpermute; `addr` = 4 * (lane ^ mask).
__device__ __forceinline__ float shfl_xor_f(float v, int addr)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double shfl_xor_f(double v, int addr)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// 2x2 on lane bit t: each lane computes its own output from its amplitude
// and its partner's (lane ^ 2^t).
template <int R, int CTRL, typename V>
__device__ __forceinline__ void oneq_lane(int t, int lane, V (&a)[1 << R], V m00, V m01, V m10, V m11,
                                          uint32_t creg, uint32_t cval, bool tok)
{
    const bool hi = (lane >> t) & 1;
    const V ms = csel(hi, m11, m00);
    const V mo = csel(hi, m10, m01);
    const int addr = (lane ^ (1 << t)) << 2;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (CTRL < 2 || ((uint32_t)j & creg) == cval) {
            V p;
            p.x = shfl_xor_f(a[j].x, addr);
            p.y = shfl_xor_f(a[j].y, addr);
            const V y = cdot2(ms, a[j], mo, p);
            put_reg(a[j], CTRL ? csel(tok, y, a[j]) : y);
        }
    });
    pin_tile(a);
}

// Value of lane ^ 2^BIT, BIT < 4: DPP moves inside a row of 16 lanes (quad
// permutes; a mirrored half row, ^ 7, and a reversed quad, ^ 3; a rotation by
// 8), which cost one or two vector moves, no LDS traffic and no wait (bit 2
// was an LDS permute: 0.27 -> 0.24 us a complex64 operation at 13 qubits).
template <int BIT>
__device__ __forceinline__ int lane_xor_i(int v)
{
    if constexpr (BIT == 0) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);
    else if constexpr (BIT == 1) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);
    else if constexpr (BIT == 3) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);
    else return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
}
template <int BIT>
__device__ __forceinline__ float lane_xor(float v)
{
    return __int_as_float(lane_xor_i<BIT>(__float_as_int(v)));
}
template <int BIT>
__device__ __forceinline__ double lane_xor(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = lane_xor_i<BIT>((int)(b & 0xffffffffll));
    const int hi = lane_xor_i<BIT>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Exchanges the odd rows (of 16 lanes, BIT = 4, or 32, BIT = 5) of x with the
// even rows of y, in place.
template <int BIT>
__device__ __forceinline__ void swap_rows(uint32_t& x, uint32_t& y)
{
    if constexpr (BIT == 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    }
}
template <int BIT>
__device__ __forceinline__ void swap_rows(float& x, float& y)
{
    uint32_t a = __float_as_uint(x), b = __float_as_uint(y);
    swap_rows<BIT>(a, b);
    x = __uint_as_float(a);
    y = __uint_as_float(b);
}
template <int BIT>
__device__ __forceinline__ void swap_rows(double& x, double& y)
{
    const unsigned long long p = (unsigned long long)__double_as_longlong(x),
                             q = (unsigned long long)__double_as_longlong(y);
    uint32_t pl = (uint32_t)p, ph = (uint32_t)(p >> 32), ql = (uint32_t)q, qh = (uint32_t)(q >> 32);
    swap_rows<BIT>(pl, ql);
    swap_rows<BIT>(ph, qh);
    x = __longlong_as_double((long long)((unsigned long long)ph << 32 | pl));
    y = __longlong_as_double((long long)((unsigned long long)qh << 32 | ql));
}

// Exact X on lane bit BIT: each lane takes its partner's amplitude.  CTRL as
// in xgate_reg_b.  Bits 4 and 5: two slots swap rows twice, the second time in
// the other order, which leaves each slot's exchanged rows in the other one.
// With an LDS permute for every word a CX from a register bit and from a lane
// onto a lane took 0.64 and 0.74 us in complex128 at 20 qubits, now 0.36 and
// 0.52; in complex64 0.32 and 0.42, now 0.28 and 0.34.
template <int BIT, int R, int CTRL, typename V>
__device__ __forceinline__ void xgate_lane_b(V (&a)[1 << R], uint32_t creg, uint32_t cval, bool tok)
{
    auto take = [&](V& x, const V p, uint32_t j) {
        x = CTRL ? csel(CTRL < 2 ? tok : tok && (j & creg) == cval, p, x) : p;
    };
    if constexpr (BIT < 4) {
        sfor<(1 << R)>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            V p;
            p.x = lane_xor<BIT>(a[j].x);
            p.y = lane_xor<BIT>(a[j].y);
            take(a[j], p, j);
        });
    } else {
        sfor<(1 << R) / 2>([&](auto jc) {
            constexpr int j = 2 * decltype(jc)::value;
            V p = a[j], q = a[j + 1];
            swap_rows<BIT>(p.x, q.x);
            swap_rows<BIT>(p.y, q.y);
            swap_rows<BIT>(q.x, p.x);
            swap_rows<BIT>(q.y, p.y);
            take(a[j], q, j);
            take(a[j + 1], p, j + 1);
        });
    }
    pin_tile(a);
}

// Scaled form of a 2x2 on lane bit 4 or 5.  The two slots of a pair (register
// bit 0) swap rows, so that one holds the amplitudes with the bit 0 of both
// and the other those with the bit 1: then it is shear_reg_b with the same
// coefficients for every lane, and the rows are swapped back: two vector
// instructions a pair and word where each slot had an LDS permute and its wait.
// A u3 and a CZ on bits 4 and 5, mean of the two: complex128 0.34 -> 0.25 us at
// 13 qubits and 21.0 -> 14.7 us at 26; complex64 0.29 -> 0.23 us and, at 27
// qubits, 20.7 -> 17.2 us.
// EX: slot 0 ends as bit value 1; swapping back in the other order puts the
// amplitudes right and leaves the pair's slots exchanged (the planner's flip).
template <int BIT, int R, bool EX, int FORM, int TY, typename T, typename V>
__device__ __forceinline__ void shear_row_b(V (&a)[1 << R], T wr, T wi, T vr, T vi)
{
    sfor<(1 << R) / 2>([&](auto jc) {
        constexpr int j = 2 * decltype(jc)::value, jp = j + FORM, jq = j + 1 - FORM;
        swap_rows<BIT>(a[j].x, a[j + 1].x);
        swap_rows<BIT>(a[j].y, a[j + 1].y);
        axpy<TY>(a[jp], wr, wi, a[jq]);
        axpy<TY>(a[jq], vr, vi, a[jp]);
        swap_rows<BIT>(a[j + EX].x, a[j + 1 - EX].x);
        swap_rows<BIT>(a[j + EX].y, a[j + 1 - EX].y);
    });
    pin_tile(a);
}

// Scaled form of a 2x2 on lane bit BIT: the lane's amplitude plus W times its
// partner's (EX: the partner's plus W times its own), W = w on the lanes whose
// bit is 0, v on the others.  Half the multiply-adds of the full product; the
// diagonal left over is carried as in shear_reg_b.
template <int BIT, int R, bool EX, int TY, typename T, typename V>
__device__ __forceinline__ void shear_lane_b(int lane, V (&a)[1 << R], T wr, T wi, T vr, T vi)
{
    const bool hi = (lane >> BIT) & 1;
    const T cr = hi ? vr : wr, ci = hi ? vi : wi;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        V p;
        p.x = lane_xor<BIT>(a[j].x);
        p.y = lane_xor<BIT>(a[j].y);
        if constexpr (EX && TY == 0) {
            // p + c a into a: both products with a.x before a.x is replaced
            const T t = fmat(cr, a[j].x, p.x), u = fmat(ci, a[j].x, p.y);
            ex_tail(a[j].x, a[j].y, cr, ci, t, u);
        } else if constexpr (EX && TY == 1) {
            ex_real(a[j].x, cr, p.x);
            ex_real(a[j].y, cr, p.y);
        } else if constexpr (EX) {
            const T u = fmat(ci, a[j].x, p.y);
            ex_imag(a[j].x, a[j].y, ci, p.x, u);
        } else {
            axpy<TY>(a[j], cr, ci, p);
        }
    });
    pin_tile(a);
}

// ---------------------------------------------------------------------------
// Tile pass kernel
// ---------------------------------------------------------------------------

template <int R, int W>
struct MapState {
    uint64_t rb[R];     // physical offset of register bit b
    uint32_t lb[R];     // LDS offset of register bit b
    uint64_t tphys;     // physical offset of this thread (lane + wave bits)
    uint32_t tlds;      // LDS offset of this thread
    uint32_t map;
};

template <int R, int W>
__device__ __forceinline__ void set_map(MapState<R, W>& ms, uint32_t map, const int32_t* __restrict__ up_phys, int lane,
                                        int wave)
{
    ms.map = map;
    sfor<R>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        const int u = map_get(map, b);
        ms.rb[b] = 1ull << up_phys[u];
        ms.lb[b] = 1u << (6 + u);
    });
    uint64_t tp = (uint64_t)lane;
    uint32_t tl = (uint32_t)lane;
    sfor<W>([&](auto wc) {
        constexpr int w = decltype(wc)::value;
        const int u = map_get(map, R + w);
        if ((wave >> w) & 1) {
            tp |= 1ull << up_phys[u];
            tl |= 1u << (6 + u);
        }
    });
    ms.tphys = tp;
    ms.tlds = tl;
}

template <int R, int W>
__device__ __forceinline__ uint64_t reg_phys(const MapState<R, W>& ms, int j)
{
    uint64_t o = 0;
    sfor<R>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if (j & (1 << b)) o += ms.rb[b];
    });
    return o;
}

template <int R, int W>
__device__ __forceinline__ uint32_t reg_lds(const MapState<R, W>& ms, int j)
{
    uint32_t o = 0;
    sfor<R>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if (j & (1 << b)) o += ms.lb[b];
    });
    return o;
}

// Register bits in `flip` hold slot = bit ^ 1: slot offsets then run downwards
// from the offset of slot 0.  (Offsets are sums; they wrap as unsigned.)
template <int R, int W>
__device__ __forceinline__ void flip_map(MapState<R, W>& ms, uint32_t flip)
{
    sfor<R>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if ((flip >> b) & 1u) {
            ms.tphys += ms.rb[b];
            ms.tlds += ms.lb[b];
            ms.rb[b] = 0ull - ms.rb[b];
            ms.lb[b] = 0u - ms.lb[b];
        }
    });
}

// One tile of a register-tile pass: load, every operation of the pass,
// store.  `lds` is the work-group's exchange buffer (wave bits), `fresh`
// replaces the load by |0..0> (the first pass of a batched circuit).
template <typename T, int R, int W>
__device__ __forceinline__ void reg_tile(typename CxT<T>::V* __restrict__ st, const PassHdr* __restrict__ hp,
                                         const DevOp* __restrict__ ops, const T* __restrict__ coef, uint64_t tile,
                                         typename CxT<T>::V* lds, int lane, int wave, bool fresh)
{
    using V = typename CxT<T>::V;
    constexpr int NR = 1 << R;
    const int nops = hp->nops;
    const RegOpT<T>* __restrict__ prog = reinterpret_cast<const RegOpT<T>*>(ops + hp->op0);
    const int nruns = hp->nruns;
    const int32_t* __restrict__ up_phys = hp->up_phys;
    {
        uint64_t base = 0;
        for (int r = 0; r < nruns; ++r) {
            const uint64_t field = (tile >> hp->run_gshift[r]) & ((1ull << hp->run_len[r]) - 1ull);
            base |= field << hp->run_start[r];
        }
        MapState<R, W> ms;
        set_map<R, W>(ms, (uint32_t)hp->map0, up_phys, lane, wave);
        V a[NR];
        if (fresh) {
            sfor<NR>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const bool one = base + ms.tphys + reg_phys(ms, j) == 0;
                a[j].x = one ? (T)1 : (T)0;
                a[j].y = (T)0;
            });
        } else {
            const V* src = st + base + ms.tphys;
            sfor<NR>([&](auto jc) { a[decltype(jc)::value] = src[reg_phys(ms, decltype(jc)::value)]; });
        }
        // the next record is fetched while the current one runs (the program
        // ends with a pad record)
        RegOpT<T> next = prog[0];
        for (int i = 0; i < nops; ++i) {
            pin_tile(a);
            const RegOpT<T> op = next;
            next = prog[i + 1];
            if ((base & op.c_glob) != op.c_glob) continue;   // tile-uniform control
            const uint32_t c_lane = op.ctl & 255u, c_wave = (op.ctl >> 8) & 255u, creg = (op.ctl >> 16) & 255u,
                           cval = op.ctl >> 24;
            auto tok_of = [&]() {
                return ((uint32_t)lane & c_lane) == c_lane && ((uint32_t)wave & c_wave) == c_wave;
            };
            auto sign_of = [&]() { return tok_of() ? (T)-1 : (T)1; };   // lanes that do not match: +1
            auto phase_of = [&]() {
                const bool tok = tok_of();
                V ph;
                ph.x = tok ? op.k[0] : (T)1;
                ph.y = tok ? op.k[1] : (T)0;
                return ph;
            };
            auto tab_of = [&]() { return coef + op.coef; };
            // value of a table index bit outside the registers (enc_bit)
            auto bit_of = [&](uint32_t src) {
                return (((uint32_t)(wave << 6 | lane) >> (src & 31u)) & (src >> 5 & 1u)) |
                       ((uint32_t)(base >> (src >> 6 & 63u)) & (src >> 12 & 1u));
            };
            // table index of the bits outside the registers (flipped register bits start at 1)
            auto ithr_of = [&]() {
                uint32_t idx = (uint32_t)op.aux >> 8 & 63u;
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    if (q >= (op.aux & 255)) break;
                    idx |= bit_of((uint32_t)op.pos[q]) << q;
                }
                return idx;
            };
            // bits 0 and 1 of a table held in the record (its entries: `full`)
            auto lo_of = [&]() { return bit_of((uint32_t)op.aux & 8191u) != 0; };
            auto hi_of = [&]() { return bit_of((uint32_t)op.aux >> 13) != 0; };
            auto full = [&](V (&m)[4]) {
                if constexpr (sizeof(T) == 4) {
                    for (int e = 0; e < 4; ++e) m[e] = V{op.k[2 * e], op.k[2 * e + 1]};
                } else {
                    const double* __restrict__ more = prog[i].more;
                    m[0] = V{op.k[0], op.k[1]};
                    m[1] = V{op.k[2], op.k[3]};
                    m[2] = V{more[0], more[1]};
                    m[3] = V{more[2], more[3]};
                }
            };
#define QOPS_CASE_IF(CODE, COND, BODY)                                                                       \
    case CODE:                                                                                               \
        if constexpr (COND) {                                                                                \
            BODY;                                                                                            \
        } else                                                                                               \
            __builtin_unreachable();                                                                         \
        break;
#define QOPS_1Q_CASES(B, C)                                                                                  \
    QOPS_CASE_IF(RC_X_REG + 3 * B + C, (B < R), (xgate_reg_b<B, R, C>(a, creg, cval, C ? tok_of() : true)))  \
    QOPS_CASE_IF(RC_1Q_REG + 3 * B + C, (B < R), V m[4]; full(m);                                            \
                 (oneq_reg_b<B, R, C>(a, m[0], m[1], m[2], m[3], creg, cval, C ? tok_of() : true)))
#define QOPS_SHEAR_CASE(B, F, TY)                                                                            \
    QOPS_CASE_IF(RC_SHEAR_REG + 6 * B + 3 * F + TY, (B < R),                                                 \
                 (shear_reg_b<B, R, F, TY>(a, op.k[0], op.k[1], op.k[2], op.k[3])))
#define QOPS_BIT_CASES(B)                                                                                    \
    QOPS_1Q_CASES(B, 0) QOPS_1Q_CASES(B, 1) QOPS_1Q_CASES(B, 2)                                              \
    QOPS_SHEAR_CASE(B, 0, 0) QOPS_SHEAR_CASE(B, 0, 1) QOPS_SHEAR_CASE(B, 0, 2)                               \
    QOPS_SHEAR_CASE(B, 1, 0) QOPS_SHEAR_CASE(B, 1, 1) QOPS_SHEAR_CASE(B, 1, 2)                               \
    QOPS_COND_CASES((B < R), RC_SIGN1 + 2 * B, RC_PHASE1 + 2 * B, 1u << B, 0u)                               \
    QOPS_COND_CASES((B < R), RC_SIGN1 + 2 * B + 1, RC_PHASE1 + 2 * B + 1, 1u << B, 1u << B)                  \
    QOPS_CASE_IF(RC_DIAG1 + B, (B < R), (diag_regs<T, R, 1u << B, 0u>(a, tab_of(), ithr_of(), op.aux)))      \
    QOPS_CASE_IF(RC_TAB1 + B, (B < R), V m[4]; full(m); const bool lo = lo_of();                             \
                 const V p0 = csel(lo, m[1], m[0]); const V p1 = csel(lo, m[3], m[2]);                       \
                 (mul_slots<R, 1u << B, 0u>(a, p0, p1, p0, p1)))
#define QOPS_COND_CASES(COND, SIGN, PHASE, M, VAL)                                                           \
    QOPS_CASE_IF(SIGN, COND, (sign_slots<R, M, VAL>(a, sign_of())))                                          \
    QOPS_CASE_IF(PHASE, COND, (phase_slots<R, M, VAL>(a, phase_of())))
#define QOPS_PAIR_CASES(B, C)                                                                                \
    QOPS_PAIR_VALUE(B, C, 0) QOPS_PAIR_VALUE(B, C, 1) QOPS_PAIR_VALUE(B, C, 2) QOPS_PAIR_VALUE(B, C, 3)      \
    QOPS_CASE_IF(RC_DIAG2 + C * (C - 1) / 2 + B, (C < R),                                                    \
                 (diag_regs<T, R, 1u << B, 1u << C>(a, tab_of(), ithr_of(), op.aux)))                        \
    QOPS_CASE_IF(RC_TAB2 + C * (C - 1) / 2 + B, (C < R), V m[4]; full(m);                                    \
                 (mul_slots<R, 1u << B, 1u << C>(a, m[0], m[1], m[2], m[3])))                                \
    QOPS_CX_CASE(B, C, 0) QOPS_CX_CASE(B, C, 1)
#define QOPS_PAIR_VALUE(B, C, P)                                                                             \
    QOPS_COND_CASES((C < R), RC_SIGN2 + 4 * (C * (C - 1) / 2 + B) + P,                                       \
                    RC_PHASE2 + 4 * (C * (C - 1) / 2 + B) + P, (1u << B | 1u << C),                          \
                    ((P & 1 ? 1u << B : 0u) | (P & 2 ? 1u << C : 0u)))
#define QOPS_CX_CASE(B, C, P)                                                                                \
    QOPS_CASE_IF(RC_CX_REG + 2 * (2 * (C * (C - 1) / 2 + B)) + P, (C < R),                                   \
                 (cx_slots<B, R, 1u << C, P ? 1u << C : 0u>(a)))                                             \
    QOPS_CASE_IF(RC_CX_REG + 2 * (2 * (C * (C - 1) / 2 + B) + 1) + P, (C < R),                               \
                 (cx_slots<C, R, 1u << B, P ? 1u << B : 0u>(a)))
#define QOPS_LANE_CASE(B, EX, TY)                                                                            \
    QOPS_CASE_IF(RC_SHEAR_LANE + 6 * B + 3 * EX + TY, true,                                                  \
                 (shear_lane_b<B, R, EX != 0, TY>(lane, a, op.k[0], op.k[1], op.k[2], op.k[3])))
#define QOPS_LANE_CASES(B)                                                                                   \
    QOPS_LANE_CASE(B, 0, 0) QOPS_LANE_CASE(B, 0, 1) QOPS_LANE_CASE(B, 0, 2)                                  \
    QOPS_LANE_CASE(B, 1, 0) QOPS_LANE_CASE(B, 1, 1) QOPS_LANE_CASE(B, 1, 2)
#define QOPS_X_LANE(B)                                                                                       \
    QOPS_CASE_IF(RC_X_LANE + 3 * B, true, (xgate_lane_b<B, R, 0>(a, creg, cval, true)))                      \
    QOPS_CASE_IF(RC_X_LANE + 3 * B + 1, true, (xgate_lane_b<B, R, 1>(a, creg, cval, tok_of())))              \
    QOPS_CASE_IF(RC_X_LANE + 3 * B + 2, true, (xgate_lane_b<B, R, 2>(a, creg, cval, tok_of())))
#define QOPS_ROW_CASE(B, EX, F, TY)                                                                          \
    QOPS_CASE_IF(RC_SHEAR_ROW + 12 * (B - 4) + 6 * EX + 3 * F + TY, true,                                    \
                 (shear_row_b<B, R, EX != 0, F, TY>(a, op.k[0], op.k[1], op.k[2], op.k[3])))
#define QOPS_ROW_CASES(B, EX)                                                                                \
    QOPS_ROW_CASE(B, EX, 0, 0) QOPS_ROW_CASE(B, EX, 0, 1) QOPS_ROW_CASE(B, EX, 0, 2)                         \
    QOPS_ROW_CASE(B, EX, 1, 0) QOPS_ROW_CASE(B, EX, 1, 1) QOPS_ROW_CASE(B, EX, 1, 2)
#define QOPS_LANE_1Q(C)                                                                                      \
    QOPS_CASE_IF(RC_1Q_LANE + C, true, V m[4]; full(m);                                                      \
                 (oneq_lane<R, C>(op.aux, lane, a, m[0], m[1], m[2], m[3], creg, cval, C ? tok_of() : true)))
            switch (op.code) {
            QOPS_BIT_CASES(0) QOPS_BIT_CASES(1) QOPS_BIT_CASES(2) QOPS_BIT_CASES(3) QOPS_BIT_CASES(4)
            QOPS_PAIR_CASES(0, 1) QOPS_PAIR_CASES(0, 2) QOPS_PAIR_CASES(1, 2) QOPS_PAIR_CASES(0, 3)
            QOPS_PAIR_CASES(1, 3) QOPS_PAIR_CASES(2, 3) QOPS_PAIR_CASES(0, 4) QOPS_PAIR_CASES(1, 4)
            QOPS_PAIR_CASES(2, 4) QOPS_PAIR_CASES(3, 4)
            QOPS_LANE_CASES(0) QOPS_LANE_CASES(1) QOPS_LANE_CASES(2)
            QOPS_LANE_CASES(3)
            QOPS_ROW_CASES(4, 0) QOPS_ROW_CASES(4, 1) QOPS_ROW_CASES(5, 0) QOPS_ROW_CASES(5, 1)
            QOPS_LANE_1Q(0) QOPS_LANE_1Q(1) QOPS_LANE_1Q(2)
            QOPS_X_LANE(0) QOPS_X_LANE(1) QOPS_X_LANE(2) QOPS_X_LANE(3) QOPS_X_LANE(4) QOPS_X_LANE(5)
            QOPS_COND_CASES(true, RC_SIGN0, RC_PHASE0, 0u, 0u)
            QOPS_CASE_IF(RC_DIAG0, true, (phase_slots<R, 0u, 0u>(a, ldc(tab_of(), (int)ithr_of()))))
            QOPS_CASE_IF(RC_TAB0, true, V m[4]; full(m); const bool lo = lo_of();
                         (phase_slots<R, 0u, 0u>(a, csel(hi_of(), csel(lo, m[3], m[2]), csel(lo, m[1], m[0])))))
            case RC_SIGN: {
                const T sgn = sign_of();
                sfor<NR>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    if (((uint32_t)j & creg) == cval) {
                        a[j].x *= sgn;
                        a[j].y *= sgn;
                    }
                });
                pin_tile(a);
                break;
            }
            case RC_PHASE: {
                const V ph = phase_of();
                sfor<NR>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    if (((uint32_t)j & creg) == cval) cmul_to(a[j], ph);
                });
                pin_tile(a);
                break;
            }
            case RC_DIAG: {
                const T* tab = tab_of();
                const uint32_t ithr = ithr_of();
                uint32_t off[NR];       // index bits that differ from slot 0's
                off[0] = 0;
                sfor<NR>([&](auto jc) {
                    constexpr uint32_t j = decltype(jc)::value;
                    if constexpr (j > 0) off[j] = off[j & (j - 1)] ^ (op.ctl >> 8 * __builtin_ctz(j) & 63u);
                });
                sfor<NR>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    cmul_to(a[j], ldc(tab, (int)(ithr ^ off[j])));
                });
                pin_tile(a);
                break;
            }
            case RC_REMAP: {
                flip_map<R, W>(ms, creg);
                __syncthreads();
                sfor<NR>([&](auto jc) { lds[ms.tlds + reg_lds(ms, decltype(jc)::value)] = a[decltype(jc)::value]; });
                __syncthreads();
                set_map<R, W>(ms, (uint32_t)op.aux, up_phys, lane, wave);
                sfor<NR>([&](auto jc) { a[decltype(jc)::value] = lds[ms.tlds + reg_lds(ms, decltype(jc)::value)]; });
                pin_tile(a);
                break;
            }
            default:
                __builtin_unreachable();
            }
        }
        {
            // an opaque copy of the thread offset keeps the compiler from
            // holding every load address live across the operation loop
            flip_map<R, W>(ms, (uint32_t)hp->flip);
            uint64_t tp = ms.tphys;
            asm volatile("" : "+v"(tp));
            V* dst = st + base + tp;
            const T sc = (T)hp->scale;
            sfor<NR>([&](auto jc) {
                V w = a[decltype(jc)::value];
                w.x *= sc;
                w.y *= sc;
                dst[reg_phys(ms, decltype(jc)::value)] = w;
            });
        }
    }
}

// Tile numbers (single circuit) or (circuit, tile) items (batched executor:
// pass `pass` of every circuit in `items`, all planned with this split), in a
// grid-stride loop.  One kernel for both, as the body is most of the code.
template <typename T, int R, int W>
__global__ void __launch_bounds__(64 << W)
tile_pass_kernel(typename CxT<T>::V* __restrict__ state, const PassHdr* __restrict__ hdrs, const DevOp* __restrict__ ops,
                 const T* __restrict__ coef, uint64_t count, const BatchItem* __restrict__ items,
                 const BatchCirc* __restrict__ circs, int pass)
{
    using V = typename CxT<T>::V;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V* lds = reinterpret_cast<V*>(smem_raw);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    for (uint64_t i = blockIdx.x; i < count; i += gridDim.x) {
        V* st = state;
        int hdr = 0;            // the pass (single circuit) or its place among the batch's headers
        uint64_t tile = i;
        if (items) {
            const BatchItem it = items[i];
            st = reinterpret_cast<V*>(circs[it.c].state);
            hdr = circs[it.c].hdr0 + pass;
            tile = (uint64_t)it.tile;
        }
        reg_tile<T, R, W>(st, hdrs + hdr, ops, coef, tile, lds, lane, wave, items && pass == 0);
    }
}

template <typename T, int R, int W>
static hipError_t launch_reg(void* state, const PassHdr* hdrs, const DevOp* ops, const void* coef, uint64_t count,
                             const BatchItem* items, const BatchCirc* circs, int pass, uint64_t grid, int lds_bytes,
                             hipStream_t s)
{
    auto fn = tile_pass_kernel<T, R, W>;
    // dynamic LDS beyond 64 KiB has to be allowed (per device)
    if (lds_bytes > 64 * 1024)
        if (hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes))
            return e;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(64 << W), lds_bytes, s,
                       reinterpret_cast<typename CxT<T>::V*>(state), hdrs, ops, reinterpret_cast<const T*>(coef), count,
                       items, circs, pass);
    return hipGetLastError();
}

template <typename T, int R, int W>
hipError_t launch_tile_t(void* state, const PassHdr* hdr, const DevOp* ops, const void* coef, uint64_t ntiles,
                         int lds_bytes, int grid_cap, hipStream_t s)
{
    uint64_t grid = ntiles;
    if (grid_cap > 0 && grid > (uint64_t)grid_cap) grid = (uint64_t)grid_cap;
    if (grid > 0x7fffffffull) grid = 0x7fffffffull;
    return launch_reg<T, R, W>(state, hdr, ops, coef, ntiles, nullptr, nullptr, 0, grid, lds_bytes, s);
}

template <typename T, int R, int W>
hipError_t launch_batch_reg_t(const BatchItem* items, int nitems, const BatchCirc* circs, const PassHdr* hdrs,
                              const DevOp* ops, const void* coef, int pass, int lds_bytes, int grid, hipStream_t s)
{
    return launch_reg<T, R, W>(nullptr, hdrs, ops, coef, (uint64_t)nitems, items, circs, pass,
                               (uint64_t)std::max(1, std::min(nitems, grid)), lds_bytes, s);
}

template hipError_t launch_tile_t<QOPS_RT_T, QOPS_RT_R, QOPS_RT_W>(void*, const PassHdr*, const DevOp*, const void*,
                                                                   uint64_t, int, int, hipStream_t);
template hipError_t launch_batch_reg_t<QOPS_RT_T, QOPS_RT_R, QOPS_RT_W>(const BatchItem*, int, const BatchCirc*,
                                                                        const PassHdr*, const DevOp*, const void*,
                                                                        int, int, int, hipStream_t);

}  // namespace qops

#else   // dispatch

namespace qops {

hipError_t launch_tile_pass(int prec, int R, int W, void* state, const PassHdr* hdr, const DevOp* ops,
                            const void* coef, uint64_t ntiles, int lds_bytes, int grid_cap, hipStream_t s)
{
#define QOPS_LAUNCH(r, w)                                                                              \
    if (R == r && W == w)                                                                              \
        return prec == 0 ? launch_tile_t<float, r, w>(state, hdr, ops, coef, ntiles, lds_bytes, grid_cap, s) \
                         : launch_tile_t<double, r, w>(state, hdr, ops, coef, ntiles, lds_bytes, grid_cap, s);
    QOPS_TILE_VARIANTS(QOPS_LAUNCH)
#undef QOPS_LAUNCH
    return hipErrorInvalidValue;
}

hipError_t launch_batch_reg(int prec, int R, int W, const BatchItem* items, int nitems, const BatchCirc* circs,
                            const PassHdr* hdrs, const DevOp* ops, const void* coef, int pass, int lds_bytes,
                            int grid, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
#define QOPS_LAUNCH(r, w)                                                                                      \
    if (R == r && W == w)                                                                                      \
        return prec == 0 ? launch_batch_reg_t<float, r, w>(items, nitems, circs, hdrs, ops, coef, pass, lds_bytes,  \
                                                           grid, s)                                           \
                         : launch_batch_reg_t<double, r, w>(items, nitems, circs, hdrs, ops, coef, pass, lds_bytes, \
                                                            grid, s);
    QOPS_TILE_VARIANTS(QOPS_LAUNCH)
#undef QOPS_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace qops

#endif
