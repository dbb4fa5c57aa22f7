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

__device__ __forceinline__ void put_one(float& d, float v) { asm("v_mov_b32 %0, %1" : "=v"(d) : "v"(v)); }
__device__ __forceinline__ void put_one(double& d, double v) { asm("v_mov_b64 %0, %1" : "=v"(d) : "v"(v)); }

// a *= b (complex), in place.
template <typename V>
__device__ __forceinline__ void cmul_to(V& a, const V b)
{
    const auto t = a.y * b.y;
    const auto u = a.y * b.x;
    a.y = fmat(a.x, b.y, u);
    a.x = fmat(a.x, b.x, -t);
}

// 2x2 on register bit B.  Register-slot controls (slots whose bits `creg`
// equal `cval`) are compile-time per slot and uniform; `tok` is the per-lane
// control result.
// Exact X on register bit B: exchange the two halves (no arithmetic).
template <int B, int R, bool CTRL, typename V>
__device__ __forceinline__ void xgate_reg_b(V (&a)[1 << R], uint32_t creg, uint32_t cval, bool tok)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int j1 = j | (1 << B);
            if (!CTRL || ((uint32_t)j & creg) == cval) {
                const V x0 = a[j], x1 = a[j1];
                if (CTRL) {
                    a[j] = csel(tok, x1, x0);
                    a[j1] = csel(tok, x0, x1);
                } else {
                    swap_reg(a[j].x, a[j1].x);
                    swap_reg(a[j].y, a[j1].y);
                }
            }
        }
    });
    pin_tile(a);
}

template <int R, bool CTRL, typename V>
__device__ __forceinline__ void xgate_reg(int b, V (&a)[1 << R], uint32_t creg, uint32_t cval, bool tok)
{
    switch (b) {
    case 0: xgate_reg_b<0, R, CTRL>(a, creg, cval, tok); break;
    case 1: if constexpr (R > 1) xgate_reg_b<1, R, CTRL>(a, creg, cval, tok); break;
    case 2: if constexpr (R > 2) xgate_reg_b<2, R, CTRL>(a, creg, cval, tok); break;
    case 3: if constexpr (R > 3) xgate_reg_b<3, R, CTRL>(a, creg, cval, tok); break;
    case 4: if constexpr (R > 4) xgate_reg_b<4, R, CTRL>(a, creg, cval, tok); break;
    case 5: if constexpr (R > 5) xgate_reg_b<5, R, CTRL>(a, creg, cval, tok); break;
    default: __builtin_unreachable();
    }
}

template <int B, int R, bool CTRL, typename V>
__device__ __forceinline__ void oneq_reg_b(V (&a)[1 << R], V m00, V m01, V m10, V m11, uint32_t creg, uint32_t cval, bool tok)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int j1 = j | (1 << B);
            if (!CTRL || ((uint32_t)j & creg) == cval) {
                const V x0 = a[j], x1 = a[j1];
                const V y0 = cdot2(m00, x0, m01, x1);
                const V y1 = cdot2(m10, x0, m11, x1);
                if (CTRL) {
                    a[j] = csel(tok, y0, x0);
                    a[j1] = csel(tok, y1, x1);
                } else {
                    put_reg(a[j], y0);
                    put_reg(a[j1], y1);
                }
            }
        }
    });
    pin_tile(a);
}

template <int R, bool CTRL, typename V>
__device__ __forceinline__ void oneq_reg(int b, V (&a)[1 << R], V m00, V m01, V m10, V m11, uint32_t creg, uint32_t cval, bool tok)
{
    switch (b) {
    case 0: oneq_reg_b<0, R, CTRL>(a, m00, m01, m10, m11, creg, cval, tok); break;
    case 1: if constexpr (R > 1) oneq_reg_b<1, R, CTRL>(a, m00, m01, m10, m11, creg, cval, tok); break;
    case 2: if constexpr (R > 2) oneq_reg_b<2, R, CTRL>(a, m00, m01, m10, m11, creg, cval, tok); break;
    case 3: if constexpr (R > 3) oneq_reg_b<3, R, CTRL>(a, m00, m01, m10, m11, creg, cval, tok); break;
    case 4: if constexpr (R > 4) oneq_reg_b<4, R, CTRL>(a, m00, m01, m10, m11, creg, cval, tok); break;
    case 5: if constexpr (R > 5) oneq_reg_b<5, R, CTRL>(a, m00, m01, m10, m11, creg, cval, tok); break;
    default: __builtin_unreachable();
    }
}

// Two-step (sheared) form of a 2x2 on register bit B: p += w q, then
// q += v p, with p the slots whose bit is FORM (0 or 1) and q the others.
// The 2x2 it stands for is diag(d0, d1) times this, possibly with the two
// slots exchanged; the planner carries the diagonal into the next operation
// on that bit and the exchange into the slot's index (DevOp::c_tile,
// PassHdr::flip).  Both steps update in place: 4 fused multiply-adds per
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

template <int R, int FORM, int TY, typename T, typename V>
__device__ __forceinline__ void shear_reg(int b, V (&a)[1 << R], T wr, T wi, T vr, T vi)
{
    switch (b) {
    case 0: shear_reg_b<0, R, FORM, TY>(a, wr, wi, vr, vi); break;
    case 1: if constexpr (R > 1) shear_reg_b<1, R, FORM, TY>(a, wr, wi, vr, vi); break;
    case 2: if constexpr (R > 2) shear_reg_b<2, R, FORM, TY>(a, wr, wi, vr, vi); break;
    case 3: if constexpr (R > 3) shear_reg_b<3, R, FORM, TY>(a, wr, wi, vr, vi); break;
    case 4: if constexpr (R > 4) shear_reg_b<4, R, FORM, TY>(a, wr, wi, vr, vi); break;
    case 5: if constexpr (R > 5) shear_reg_b<5, R, FORM, TY>(a, wr, wi, vr, vi); break;
    default: __builtin_unreachable();
    }
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

// Exact X on lane bit t: take the partner's amplitude.
template <int R, bool CTRL, typename V>
__device__ __forceinline__ void xgate_lane(int t, int lane, V (&a)[1 << R], uint32_t creg, uint32_t cval, bool tok)
{
    const int addr = (lane ^ (1 << t)) << 2;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (!CTRL || ((uint32_t)j & creg) == cval) {
            V p;
            p.x = shfl_xor_f(a[j].x, addr);
            p.y = shfl_xor_f(a[j].y, addr);
            a[j] = CTRL ? csel(tok, p, a[j]) : p;
        }
    });
    pin_tile(a);
}

// 2x2 on lane bit t: each lane computes its own output from its amplitude
// and its partner's (lane ^ 2^t).
template <int R, bool CTRL, typename V>
__device__ __forceinline__ void oneq_lane(int t, int lane, V (&a)[1 << R], V m00, V m01, V m10, V m11,
                                          uint32_t creg, uint32_t cval, bool tok)
{
    const bool hi = (lane >> t) & 1;
    const V ms = csel(hi, m11, m00);
    const V mo = csel(hi, m10, m01);
    const int addr = (lane ^ (1 << t)) << 2;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (!CTRL || ((uint32_t)j & creg) == cval) {
            V p;
            p.x = shfl_xor_f(a[j].x, addr);
            p.y = shfl_xor_f(a[j].y, addr);
            const V y = cdot2(ms, a[j], mo, p);
            if (CTRL)
                a[j] = csel(tok, y, a[j]);
            else
                put_reg(a[j], y);
        }
    });
    pin_tile(a);
}

// Value of lane ^ 2^BIT.  Bits 0, 1 and 3 are DPP moves inside a row of 16
// lanes (quad permutes; a rotation by 8), which cost one vector move and no
// LDS traffic; the others go through ds_bpermute.
template <int BIT>
__device__ __forceinline__ int lane_xor_i(int v, int addr)
{
    if constexpr (BIT == 0) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);
    else if constexpr (BIT == 1) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);
    else if constexpr (BIT == 3) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true);
    else return __builtin_amdgcn_ds_bpermute(addr, v);
}
template <int BIT>
__device__ __forceinline__ float lane_xor(float v, int addr)
{
    return __int_as_float(lane_xor_i<BIT>(__float_as_int(v), addr));
}
template <int BIT>
__device__ __forceinline__ double lane_xor(double v, int addr)
{
    const long long b = __double_as_longlong(v);
    const int lo = lane_xor_i<BIT>((int)(b & 0xffffffffll), addr);
    const int hi = lane_xor_i<BIT>((int)(b >> 32), addr);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
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
    const int addr = (lane ^ (1 << BIT)) << 2;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        V p;
        p.x = lane_xor<BIT>(a[j].x, addr);
        p.y = lane_xor<BIT>(a[j].y, addr);
        if constexpr (EX && TY == 0) {
            // p + c a into a: both products with a.x before a.x is replaced
            const T t = fmat(cr, a[j].x, p.x), u = fmat(ci, a[j].x, p.y);
            a[j].x = fmat(-ci, a[j].y, t);
            a[j].y = fmat(cr, a[j].y, u);
        } else if constexpr (EX && TY == 1) {
            a[j].x = fmat(cr, a[j].x, p.x);
            a[j].y = fmat(cr, a[j].y, p.y);
        } else if constexpr (EX) {
            const T u = fmat(ci, a[j].x, p.y);
            a[j].x = fmat(-ci, a[j].y, p.x);
            put_one(a[j].y, u);
        } else {
            axpy<TY>(a[j], cr, ci, p);
        }
    });
    pin_tile(a);
}

template <int R, bool EX, int TY, typename T, typename V>
__device__ __forceinline__ void shear_lane(int t, int lane, V (&a)[1 << R], T wr, T wi, T vr, T vi)
{
    switch (t) {
    case 0: shear_lane_b<0, R, EX, TY>(lane, a, wr, wi, vr, vi); break;
    case 1: shear_lane_b<1, R, EX, TY>(lane, a, wr, wi, vr, vi); break;
    case 2: shear_lane_b<2, R, EX, TY>(lane, a, wr, wi, vr, vi); break;
    case 3: shear_lane_b<3, R, EX, TY>(lane, a, wr, wi, vr, vi); break;
    case 4: shear_lane_b<4, R, EX, TY>(lane, a, wr, wi, vr, vi); break;
    case 5: shear_lane_b<5, R, EX, TY>(lane, a, wr, wi, vr, vi); break;
    default: __builtin_unreachable();
    }
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
    const DevOp* __restrict__ prog = ops + hp->op0;
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
        for (int i = 0; i < nops; ++i) {
            pin_tile(a);
            const DevOp op = prog[i];
            if ((base & op.c_glob) != op.c_glob) continue;   // tile-uniform control
            switch (op.type) {
            case OP_SHEAR_REG: {
                const T* c = coef + op.coef;
                const T wr = c[0], wi = c[1], vr = c[2], vi = c[3];
                if (op.b == 0) {
                    if (op.c_lane == 0) shear_reg<R, 0, 0>(op.a, a, wr, wi, vr, vi);
                    else if (op.c_lane == 1) shear_reg<R, 0, 1>(op.a, a, wr, wi, vr, vi);
                    else shear_reg<R, 0, 2>(op.a, a, wr, wi, vr, vi);
                } else {
                    if (op.c_lane == 0) shear_reg<R, 1, 0>(op.a, a, wr, wi, vr, vi);
                    else if (op.c_lane == 1) shear_reg<R, 1, 1>(op.a, a, wr, wi, vr, vi);
                    else shear_reg<R, 1, 2>(op.a, a, wr, wi, vr, vi);
                }
                break;
            }
            case OP_SHEAR_LANE: {
                const T* c = coef + op.coef;
                const T wr = c[0], wi = c[1], vr = c[2], vi = c[3];
                if (op.b == 0) {
                    if (op.c_lane == 0) shear_lane<R, false, 0>(op.a, lane, a, wr, wi, vr, vi);
                    else if (op.c_lane == 1) shear_lane<R, false, 1>(op.a, lane, a, wr, wi, vr, vi);
                    else shear_lane<R, false, 2>(op.a, lane, a, wr, wi, vr, vi);
                } else {
                    if (op.c_lane == 0) shear_lane<R, true, 0>(op.a, lane, a, wr, wi, vr, vi);
                    else if (op.c_lane == 1) shear_lane<R, true, 1>(op.a, lane, a, wr, wi, vr, vi);
                    else shear_lane<R, true, 2>(op.a, lane, a, wr, wi, vr, vi);
                }
                break;
            }
            case OP_1Q_REG:
            case OP_1Q_LANE: {
                const T* c = coef + op.coef;
                const V m00 = ldc(c, 0), m01 = ldc(c, 1), m10 = ldc(c, 2), m11 = ldc(c, 3);
                const bool ctrl = (op.c_lane | op.c_wave | op.c_reg) != 0;
                const bool tok = ((uint32_t)lane & op.c_lane) == op.c_lane && ((uint32_t)wave & op.c_wave) == op.c_wave;
                if (op.b == 1) {   // exact X: exchange only
                    if (op.type == OP_1Q_REG) {
                        if (ctrl) xgate_reg<R, true>(op.a, a, op.c_reg, op.c_tile, tok);
                        else xgate_reg<R, false>(op.a, a, 0u, 0u, true);
                    } else {
                        if (ctrl) xgate_lane<R, true>(op.a, lane, a, op.c_reg, op.c_tile, tok);
                        else xgate_lane<R, false>(op.a, lane, a, 0u, 0u, true);
                    }
                } else if (op.type == OP_1Q_REG) {
                    if (ctrl)
                        oneq_reg<R, true>(op.a, a, m00, m01, m10, m11, op.c_reg, op.c_tile, tok);
                    else
                        oneq_reg<R, false>(op.a, a, m00, m01, m10, m11, 0u, 0u, true);
                } else {
                    if (ctrl)
                        oneq_lane<R, true>(op.a, lane, a, m00, m01, m10, m11, op.c_reg, op.c_tile, tok);
                    else
                        oneq_lane<R, false>(op.a, lane, a, m00, m01, m10, m11, 0u, 0u, true);
                }
                break;
            }
            case OP_CPHASE: {
                // phase on the amplitudes whose masked bits are all 1; the
                // register part of the condition is uniform per slot
                const bool tok = ((uint32_t)lane & op.c_lane) == op.c_lane && ((uint32_t)wave & op.c_wave) == op.c_wave;
                const bool thr = (op.c_lane | op.c_wave) != 0;
                const uint32_t creg = op.c_reg, cval = op.c_tile;
                // the multiplier is 1 where the lane's bits do not match
                V ph = ldc(coef + op.coef, 0);
                if (thr) {
                    ph.x = tok ? ph.x : (T)1;
                    ph.y = tok ? ph.y : (T)0;
                }
                if (op.b == 1) {   // -1: flip signs (lanes that do not match multiply by +1)
                    const T sgn = ph.x;
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if (((uint32_t)j & creg) == cval) {
                            a[j].x *= sgn;
                            a[j].y *= sgn;
                        }
                    });
                } else {
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if (((uint32_t)j & creg) == cval) cmul_to(a[j], ph);
                    });
                }
                pin_tile(a);
                break;
            }
            case OP_DIAG: {
                const T* tab = coef + op.coef;
                const int m = op.a;
                uint32_t ithr = op.c_tile;   // table bits on flipped register bits start at 1
                uint32_t rm[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    rm[q] = 0;
                    if (q < m) {
                        const int cls = op.pos[q] >> 8, v = op.pos[q] & 255;
                        if (cls == SRC_LANE) ithr |= (uint32_t)((lane >> v) & 1) << q;
                        else if (cls == SRC_WAVE) ithr |= (uint32_t)((wave >> v) & 1) << q;
                        else if (cls == SRC_GLOB) ithr |= (uint32_t)((base >> v) & 1ull) << q;
                        else rm[q] = 1u << v;
                    }
                }
                // table bits held in registers: at most two take the fast path
                // (the four candidate phases are loaded once per thread and
                // selected per slot with uniform conditions)
                int nq = 0, qa = -1, qb = -1;
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    if (rm[q]) {
                        if (nq == 0) qa = q;
                        else if (nq == 1) qb = q;
                        ++nq;
                    }
                if (nq <= 2) {
                    const uint32_t ba = qa >= 0 ? 1u << qa : 0u, bb = qb >= 0 ? 1u << qb : 0u;
                    const uint32_t ma = qa >= 0 ? rm[qa] : 0u, mb = qb >= 0 ? rm[qb] : 0u;
                    V pv[4];
                    pv[0] = ldc(tab, (int)ithr);
                    pv[1] = ldc(tab, (int)(ithr ^ ba));
                    pv[2] = ldc(tab, (int)(ithr ^ bb));
                    pv[3] = ldc(tab, (int)(ithr ^ (ba | bb)));
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const int r = (((uint32_t)j & ma) ? 1 : 0) | (((uint32_t)j & mb) ? 2 : 0);   // uniform
                        if (r == 0) cmul_to(a[j], pv[0]);
                        else if (r == 1) cmul_to(a[j], pv[1]);
                        else if (r == 2) cmul_to(a[j], pv[2]);
                        else cmul_to(a[j], pv[3]);
                    });
                } else {
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        uint32_t idx = ithr;
#pragma unroll
                        for (int q = 0; q < 6; ++q)
                            if ((uint32_t)j & rm[q]) idx ^= 1u << q;
                        cmul_to(a[j], ldc(tab, (int)idx));
                    });
                }
                pin_tile(a);
                break;
            }
            case OP_REMAP: {
                flip_map<R, W>(ms, op.c_reg);
                __syncthreads();
                sfor<NR>([&](auto jc) { lds[ms.tlds + reg_lds(ms, decltype(jc)::value)] = a[decltype(jc)::value]; });
                __syncthreads();
                set_map<R, W>(ms, (uint32_t)op.b, up_phys, lane, wave);
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

template <typename T, int R, int W>
__global__ void __launch_bounds__(64 << W)
tile_pass_kernel(typename CxT<T>::V* __restrict__ st, const PassHdr* __restrict__ hp, const DevOp* __restrict__ ops,
                 const T* __restrict__ coef, uint64_t ntiles)
{
    using V = typename CxT<T>::V;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V* lds = reinterpret_cast<V*>(smem_raw);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
        reg_tile<T, R, W>(st, hp, ops, coef, tile, lds, lane, wave, false);
}

// Batched executor: register-tile pass `pass` of every circuit in `items`
// (all planned with the same register/wave split).
template <typename T, int R, int W>
__global__ void __launch_bounds__(64 << W)
batch_reg_kernel(const BatchItem* __restrict__ items, int nitems, const BatchCirc* __restrict__ circs,
                 const PassHdr* __restrict__ hdrs, const DevOp* __restrict__ ops, const T* __restrict__ coef, int pass)
{
    using V = typename CxT<T>::V;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    V* lds = reinterpret_cast<V*>(smem_raw);
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    for (int i = blockIdx.x; i < nitems; i += gridDim.x) {
        const BatchItem it = items[i];
        const BatchCirc c = circs[it.c];
        reg_tile<T, R, W>(reinterpret_cast<V*>(c.state), hdrs + c.hdr0 + pass, ops, coef, (uint64_t)it.tile, lds,
                          lane, wave, pass == 0);
    }
}

template <typename T, int R, int W>
hipError_t launch_tile_t(void* state, const PassHdr* hdr, const DevOp* ops, const void* coef, uint64_t ntiles,
                                int lds_bytes, int grid_cap, hipStream_t s)
{
    using V = typename CxT<T>::V;
    auto fn = tile_pass_kernel<T, R, W>;
    static bool attr_done = false;
    if (!attr_done) {
        (void)hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, tile_max_lds_bytes());
        attr_done = true;
    }
    uint64_t grid = ntiles;
    if (grid_cap > 0 && grid > (uint64_t)grid_cap) grid = (uint64_t)grid_cap;
    if (grid > 0x7fffffffull) grid = 0x7fffffffull;
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(64 << W), lds_bytes, s, reinterpret_cast<V*>(state), hdr, ops,
                       reinterpret_cast<const T*>(coef), ntiles);
    return hipGetLastError();
}

template <typename T, int R, int W>
hipError_t launch_batch_reg_t(const BatchItem* items, int nitems, const BatchCirc* circs, const PassHdr* hdrs,
                                     const DevOp* ops, const void* coef, int pass, int lds_bytes, int grid,
                                     hipStream_t s)
{
    if (hipError_t e = hipFuncSetAttribute((const void*)batch_reg_kernel<T, R, W>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes))
        return e;
    const int g = std::max(1, std::min(nitems, grid));
    hipLaunchKernelGGL((batch_reg_kernel<T, R, W>), dim3(g), dim3(64 << W), lds_bytes, s, items, nitems, circs, hdrs,
                       ops, reinterpret_cast<const T*>(coef), pass);
    return hipGetLastError();
}

template hipError_t launch_tile_t<QOPS_RT_T, QOPS_RT_R, QOPS_RT_W>(void*, const PassHdr*, const DevOp*, const void*,
                                                                   uint64_t, int, int, hipStream_t);
template hipError_t launch_batch_reg_t<QOPS_RT_T, QOPS_RT_R, QOPS_RT_W>(const BatchItem*, int, const BatchCirc*,
                                                                        const PassHdr*, const DevOp*, const void*,
                                                                        int, int, int, hipStream_t);

}  // namespace qops

#else   // dispatch

namespace qops {

bool tile_variant_supported(int prec, int R, int W)
{
#define QOPS_CHECK(r, w) if (R == r && W == w) return true;
    (void)prec;
    QOPS_TILE_VARIANTS(QOPS_CHECK)
#undef QOPS_CHECK
    return false;
}

int tile_max_lds_bytes() { return 160 * 1024; }

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
