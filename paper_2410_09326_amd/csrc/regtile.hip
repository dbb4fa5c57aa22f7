// Register tile pass: a wave holds 2^(6+R) amplitudes of the state in its
// registers (2^(6+R+W) in a work-group of 2^W waves), runs every operation of
// a pass on them and writes them back.  Also the batched form of the same
// body (pass p of many circuits in one launch).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "devprog.hpp"
#include "devutil.hpp"
#include "kernels.hpp"

namespace qops {

// ---------------------------------------------------------------------------
// Register-resident operations
// ---------------------------------------------------------------------------

// 2x2 on register bit B.  Register-slot controls `creg` are compile-time per
// slot and uniform; `tok` is the per-lane control result.
// Exact X on register bit B: exchange the two halves (no arithmetic).
template <int B, int R, bool CTRL, typename V>
__device__ __forceinline__ void xgate_reg_b(V (&a)[1 << R], uint32_t creg, bool tok)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int j1 = j | (1 << B);
            if (!CTRL || ((uint32_t)j & creg) == creg) {
                const V x0 = a[j], x1 = a[j1];
                if (CTRL) {
                    a[j] = csel(tok, x1, x0);
                    a[j1] = csel(tok, x0, x1);
                } else {
                    a[j] = x1;
                    a[j1] = x0;
                }
            }
        }
    });
}

template <int R, bool CTRL, typename V>
__device__ __forceinline__ void xgate_reg(int b, V (&a)[1 << R], uint32_t creg, bool tok)
{
    switch (b) {
    case 0: xgate_reg_b<0, R, CTRL>(a, creg, tok); break;
    case 1: if constexpr (R > 1) xgate_reg_b<1, R, CTRL>(a, creg, tok); break;
    case 2: if constexpr (R > 2) xgate_reg_b<2, R, CTRL>(a, creg, tok); break;
    case 3: if constexpr (R > 3) xgate_reg_b<3, R, CTRL>(a, creg, tok); break;
    case 4: if constexpr (R > 4) xgate_reg_b<4, R, CTRL>(a, creg, tok); break;
    case 5: if constexpr (R > 5) xgate_reg_b<5, R, CTRL>(a, creg, tok); break;
    default: break;
    }
}

template <int B, int R, bool CTRL, typename V>
__device__ __forceinline__ void oneq_reg_b(V (&a)[1 << R], V m00, V m01, V m10, V m11, uint32_t creg, bool tok)
{
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (!(j & (1 << B))) {
            constexpr int j1 = j | (1 << B);
            if (!CTRL || ((uint32_t)j & creg) == creg) {
                const V x0 = a[j], x1 = a[j1];
                const V y0 = cdot2(m00, x0, m01, x1);
                const V y1 = cdot2(m10, x0, m11, x1);
                if (CTRL) {
                    a[j] = csel(tok, y0, x0);
                    a[j1] = csel(tok, y1, x1);
                } else {
                    a[j] = y0;
                    a[j1] = y1;
                }
            }
        }
    });
}

template <int R, bool CTRL, typename V>
__device__ __forceinline__ void oneq_reg(int b, V (&a)[1 << R], V m00, V m01, V m10, V m11, uint32_t creg, bool tok)
{
    switch (b) {
    case 0: oneq_reg_b<0, R, CTRL>(a, m00, m01, m10, m11, creg, tok); break;
    case 1: if constexpr (R > 1) oneq_reg_b<1, R, CTRL>(a, m00, m01, m10, m11, creg, tok); break;
    case 2: if constexpr (R > 2) oneq_reg_b<2, R, CTRL>(a, m00, m01, m10, m11, creg, tok); break;
    case 3: if constexpr (R > 3) oneq_reg_b<3, R, CTRL>(a, m00, m01, m10, m11, creg, tok); break;
    case 4: if constexpr (R > 4) oneq_reg_b<4, R, CTRL>(a, m00, m01, m10, m11, creg, tok); break;
    case 5: if constexpr (R > 5) oneq_reg_b<5, R, CTRL>(a, m00, m01, m10, m11, creg, tok); break;
    default: break;
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
__device__ __forceinline__ void xgate_lane(int t, int lane, V (&a)[1 << R], uint32_t creg, bool tok)
{
    const int addr = (lane ^ (1 << t)) << 2;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (!CTRL || ((uint32_t)j & creg) == creg) {
            V p;
            p.x = shfl_xor_f(a[j].x, addr);
            p.y = shfl_xor_f(a[j].y, addr);
            a[j] = CTRL ? csel(tok, p, a[j]) : p;
        }
    });
}

// 2x2 on lane bit t: each lane computes its own output from its amplitude
// and its partner's (lane ^ 2^t).
template <int R, bool CTRL, typename V>
__device__ __forceinline__ void oneq_lane(int t, int lane, V (&a)[1 << R], V m00, V m01, V m10, V m11,
                                          uint32_t creg, bool tok)
{
    const bool hi = (lane >> t) & 1;
    const V ms = csel(hi, m11, m00);
    const V mo = csel(hi, m10, m01);
    const int addr = (lane ^ (1 << t)) << 2;
    sfor<(1 << R)>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (!CTRL || ((uint32_t)j & creg) == creg) {
            V p;
            p.x = shfl_xor_f(a[j].x, addr);
            p.y = shfl_xor_f(a[j].y, addr);
            const V y = cdot2(ms, a[j], mo, p);
            if (CTRL)
                a[j] = csel(tok, y, a[j]);
            else
                a[j] = y;
        }
    });
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
        if (j & (1 << b)) o |= ms.rb[b];
    });
    return o;
}

template <int R, int W>
__device__ __forceinline__ uint32_t reg_lds(const MapState<R, W>& ms, int j)
{
    uint32_t o = 0;
    sfor<R>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if (j & (1 << b)) o |= ms.lb[b];
    });
    return o;
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
            const DevOp op = prog[i];
            if ((base & op.c_glob) != op.c_glob) continue;   // tile-uniform control
            switch (op.type) {
            case OP_1Q_REG:
            case OP_1Q_LANE: {
                const T* c = coef + op.coef;
                const V m00 = ldc(c, 0), m01 = ldc(c, 1), m10 = ldc(c, 2), m11 = ldc(c, 3);
                const bool ctrl = (op.c_lane | op.c_wave | op.c_reg) != 0;
                const bool tok = ((uint32_t)lane & op.c_lane) == op.c_lane && ((uint32_t)wave & op.c_wave) == op.c_wave;
                if (op.b == 1) {   // exact X: exchange only
                    if (op.type == OP_1Q_REG) {
                        if (ctrl) xgate_reg<R, true>(op.a, a, op.c_reg, tok);
                        else xgate_reg<R, false>(op.a, a, 0u, true);
                    } else {
                        if (ctrl) xgate_lane<R, true>(op.a, lane, a, op.c_reg, tok);
                        else xgate_lane<R, false>(op.a, lane, a, 0u, true);
                    }
                } else if (op.type == OP_1Q_REG) {
                    if (ctrl)
                        oneq_reg<R, true>(op.a, a, m00, m01, m10, m11, op.c_reg, tok);
                    else
                        oneq_reg<R, false>(op.a, a, m00, m01, m10, m11, 0u, true);
                } else {
                    if (ctrl)
                        oneq_lane<R, true>(op.a, lane, a, m00, m01, m10, m11, op.c_reg, tok);
                    else
                        oneq_lane<R, false>(op.a, lane, a, m00, m01, m10, m11, 0u, true);
                }
                break;
            }
            case OP_CPHASE: {
                // phase on the amplitudes whose masked bits are all 1; the
                // register part of the condition is uniform per slot
                const bool tok = ((uint32_t)lane & op.c_lane) == op.c_lane && ((uint32_t)wave & op.c_wave) == op.c_wave;
                const bool thr = (op.c_lane | op.c_wave) != 0;
                const uint32_t creg = op.c_reg;
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
                        if (((uint32_t)j & creg) == creg) {
                            a[j].x *= sgn;
                            a[j].y *= sgn;
                        }
                    });
                } else {
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if (((uint32_t)j & creg) == creg) a[j] = cmul(a[j], ph);
                    });
                }
                break;
            }
            case OP_DIAG: {
                const T* tab = coef + op.coef;
                const int m = op.a;
                uint32_t ithr = 0;
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
                    pv[1] = ldc(tab, (int)(ithr | ba));
                    pv[2] = ldc(tab, (int)(ithr | bb));
                    pv[3] = ldc(tab, (int)(ithr | ba | bb));
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const int r = (((uint32_t)j & ma) ? 1 : 0) | (((uint32_t)j & mb) ? 2 : 0);   // uniform
                        if (r == 0) a[j] = cmul(a[j], pv[0]);
                        else if (r == 1) a[j] = cmul(a[j], pv[1]);
                        else if (r == 2) a[j] = cmul(a[j], pv[2]);
                        else a[j] = cmul(a[j], pv[3]);
                    });
                } else {
                    sfor<NR>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        uint32_t idx = ithr;
#pragma unroll
                        for (int q = 0; q < 6; ++q)
                            if ((uint32_t)j & rm[q]) idx |= 1u << q;
                        a[j] = cmul(a[j], ldc(tab, (int)idx));
                    });
                }
                break;
            }
            case OP_REMAP:
            case OP_TO_LDS: {
                __syncthreads();
                sfor<NR>([&](auto jc) { lds[ms.tlds + reg_lds(ms, decltype(jc)::value)] = a[decltype(jc)::value]; });
                __syncthreads();
                if (op.type == OP_REMAP) {
                    set_map<R, W>(ms, (uint32_t)op.b, up_phys, lane, wave);
                    sfor<NR>([&](auto jc) { a[decltype(jc)::value] = lds[ms.tlds + reg_lds(ms, decltype(jc)::value)]; });
                }
                break;
            }
            case OP_FROM_LDS: {
                set_map<R, W>(ms, (uint32_t)op.b, up_phys, lane, wave);
                sfor<NR>([&](auto jc) { a[decltype(jc)::value] = lds[ms.tlds + reg_lds(ms, decltype(jc)::value)]; });
                break;
            }
            default:
                break;
            }
        }
        {
            // an opaque copy of the thread offset keeps the compiler from
            // holding every load address live across the operation loop
            uint64_t tp = ms.tphys;
            asm volatile("" : "+v"(tp));
            V* dst = st + base + tp;
            sfor<NR>([&](auto jc) { dst[reg_phys(ms, decltype(jc)::value)] = a[decltype(jc)::value]; });
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

#define QOPS_TILE_VARIANTS(X) \
    X(4, 0) X(4, 1) X(4, 2) X(5, 0) X(5, 1) X(5, 2)

bool tile_variant_supported(int prec, int R, int W)
{
#define QOPS_CHECK(r, w) if (R == r && W == w) return true;
    (void)prec;
    QOPS_TILE_VARIANTS(QOPS_CHECK)
#undef QOPS_CHECK
    return false;
}

int tile_max_lds_bytes() { return 160 * 1024; }

template <typename T, int R, int W>
static hipError_t launch_tile_t(void* state, const PassHdr* hdr, const DevOp* ops, const void* coef, uint64_t ntiles,
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

template <typename T, int R, int W>
static hipError_t launch_batch_reg_t(const BatchItem* items, int nitems, const BatchCirc* circs, const PassHdr* hdrs,
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
