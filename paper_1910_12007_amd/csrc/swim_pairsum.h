// swim_pairsum.h -- device building blocks shared by the persistent forward
// kernels (filament and full sperm model): the dense regularized-Brinkmanlet
// pair sum of eq. (BrV) in the symmetric lane schedule, the FP32 kernel
// table's LDS copy, and the compensated (hi, lo) position update.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "swim_math.h"

namespace swim {

template <typename T> struct alignas(4 * sizeof(T)) Src4 {
    T x, y, fx, fy;
};

template <typename T> struct alignas(2 * sizeof(T)) V2 {
    T x, y;
};

// The constants of one system by one wave: in T (out) and, if out64 is not
// null, in FP64 -- the values of sysconst_compute.  The scalars are lane 0's;
// coefficient n of U and of V (a sum of 40 terms each) is taken by a lane of
// its own, so that the set-up of a few systems does not wait for one thread's
// 32 sums in turn (34 us before, for any number of systems up to a thousand).
template <typename T>
__device__ inline void sysconst_wave(double alpha, double eps, SysConst<T>* out, SysConst<double>* out64, int blob,
                                     int lane)
{
    const bool pb = blob == 1 && alpha > 0.0;
    const double g0 = pb ? pb_g0_closed(alpha * eps) : 0.0;
    // the paper's blob at alpha > 0: its FP64 constants are all scalars, and
    // its FP32 ones those of the reading's blob but for H1(0) and hoff
    SysConst<double>* const p64 = sizeof(T) == 8 ? (SysConst<double>*)out : out64;
    if (pb && p64 && lane == 0) sysconst_paper<double>(alpha, eps, g0, p64);
    if (pb && sizeof(T) == 8) return;
    if (lane == 0) {
        SysConst<double> R;
        sysconst_scalars<double>(alpha, eps, &R, pb ? 0 : blob);
        if (!pb && out64) sysconst_cast_scalars<double>(R, out64);
        if (pb) {
            R.hoff = R.h1c + 0.5 * g0;
            R.h1c = -0.5 * g0;
        }
        sysconst_cast_scalars<T>(R, out);
    }
    static_assert(NT_MAX == 16, "lanes 0..15: U, lanes 16..31: V");
    if (lane < 32) {
        double v = 0.0;
        if (alpha != 0.0) {
            const double a2 = alpha * alpha, w0 = a2 * (eps * eps), L0 = log(0.25 * w0);
            const bool isU = lane < 16;
            const int n = isU ? lane + 1 : lane - 14;  // U: 1..16, V: 2..17
            double s0 = 0.0, s1 = 0.0, binom = 1.0, wp = 1.0;
#pragma unroll 4
            for (int m = 0; m < NSER_SETUP; ++m) {
                const double p0 = isU ? SETUP_SERIES.I0[m] : SETUP_SERIES.A[m];
                const double p1 = isU ? SETUP_SERIES.P0[m] : SETUP_SERIES.B[m];
                if (m >= n) {
                    s0 += binom * p0 * wp;
                    s1 += binom * p1 * wp;
                    binom = binom * (m + 1) * (1.0 / (double)(m - n + 1));
                    wp *= w0;
                }
            }
            double ap = a2;  // U: a2^n, V: a2^(n - 1)
            for (int k = 1; k < (isU ? n : n - 1); ++k) ap *= a2;
            v = (isU ? -0.5 * L0 * s0 + s1 : (n - 1) * (0.5 * L0 * s0 - s1)) * ap;
        }
        T* const o = lane < 16 ? out->U + lane : out->V + (lane - 16);
        *o = (T)v;
        if (!pb && out64) {
            double* const o64 = lane < 16 ? out64->U + lane : out64->V + (lane - 16);
            *o64 = v;
        }
    }
}

// position outside the run bound |x| <= 1e3 (or not finite)
__device__ __forceinline__ bool bad_t(float x) { return !(fabsf(x) <= 1e3f); }
__device__ __forceinline__ bool bad_t(double x) { return !(fabs(x) <= 1e3); }

// copy one system's FP32 kernel table from HBM into LDS (nthreads threads)
__device__ __forceinline__ void tab_load(const TabSys* g, TabSys* tab, int tid, int nthreads)
{
    const float4* src = reinterpret_cast<const float4*>(g);
    float4* dst = reinterpret_cast<float4*>(tab);
    constexpr int NV = (int)(sizeof(TabSys) / sizeof(float4));
    for (int i = tid; i < NV; i += nthreads) dst[i] = src[i];
}

// The FP32 table as a 64 KiB index window: the entry of index id (the bits
// of v >> TAB_SHIFT, TAB_BIAS for v = 1) sits at byte (id << 4) mod 2^15, Ht's
// coefficients there and H2's TAB_WIN_G bytes on, so the address of a pair's
// entry is (bits >> (TAB_SHIFT - 4)) & 0x7FF0: two operations, no bias and no
// clamp.  Entries 16.. of the table fill slots 0 .. TAB_N - 17, entries 0..15
// (v in [1, 2)) the last 16 slots, and every other slot is zero: the indices of
// finite v beyond the table (TAB_END .. 4079) land on zeros, as the zero entry
// TAB_N does for a clamped index.  Non-finite v (4080..4095) alias entries
// 0..15; their positions are non-finite already and end the run.  The two halves
// of an entry lie apart: a read of 16-byte pieces spreads over all banks, with
// 32-byte entries over half of them.
constexpr uint32_t TAB_WIN_BYTES = 65536, TAB_WIN_G = TAB_WIN_BYTES / 2;
static_assert(TAB_M == 4 && sizeof(TabE) == 32 && TAB_BIAS == 2032 && TAB_END <= 4080,
              "the index window holds 2048 entries of v's octaves 0..127");
__device__ __forceinline__ uint32_t tab_win_off(uint32_t bits) { return (bits >> (TAB_SHIFT - 4)) & 0x7FF0u; }

// copy one system's FP32 kernel table from HBM into its LDS index window
__device__ __forceinline__ void tab_load_window(const TabSys* g, unsigned char* win, int tid, int nthreads)
{
    const float4* src = reinterpret_cast<const float4*>(g->e);
    float4* dst = reinterpret_cast<float4*>(win);
    constexpr int HV = (int)(TAB_WIN_G / sizeof(float4)), EV = (int)(sizeof(TabE) / sizeof(float4));
    static_assert(EV == 2, "an entry is two pieces");
    for (int i = tid; i < EV * HV; i += nthreads) {
        // slot id mod 2048 holds entry id - TAB_BIAS; pieces in the table's order
        const int slot = i / EV, half = i % EV, ent = (slot - (int)TAB_BIAS) & 2047;
        dst[half * HV + slot] = ent < TAB_N ? src[ent * EV + half] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// kernel values of one FP64 pair from its system's table in HBM (the
// entries of one run, some 30 KB, stay in the caches; nine 16-byte loads per
// pair): zeros and true for a pair beyond the table
// (LDS: the table lies at that LDS address instead)
template <bool LDS = false>
__device__ __forceinline__ bool tab64_lookup(const void* tab, double t, double ts, double& Ht, double& H2,
                                             uint32_t at = 0)
{
    const double y = t * ts, v = 1.0 + y;
    const uint32_t id = tab64_index(v);
    const bool far = id >= (uint32_t)TAB_N;
    typedef double f64x2_t __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(1))) f64x2_t* GlobalD2;
    const GlobalD2 p = (GlobalD2)(uintptr_t)((const char*)tab + (size_t)min(id, (uint32_t)(TAB_N - 1)) * sizeof(TabE64));
    double c[18];
#if defined(__HIP_DEVICE_COMPILE__)
    typedef const __attribute__((address_space(3))) f64x2_t* LdsD2;
    const LdsD2 pl = (LdsD2)(uintptr_t)(at + min(id, (uint32_t)(TAB_N - 1)) * (uint32_t)sizeof(TabE64));
#else
    const GlobalD2 pl = p;
#endif
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const f64x2_t w = LDS ? pl[k] : p[k];
        c[2 * k] = w.x;
        c[2 * k + 1] = w.y;
    }
    double h, g;
    tab64_eval(c, c + 9, id, tab64_x(y, v, id), h, g);
    Ht = far ? 0.0 : h;
    H2 = far ? 0.0 : g;
    return far;
}

// direct evaluation of a pair beyond the table; not inlined, so that its
// registers (and the scalars that its hoisted coefficients take) stay out of
// the pair loops
__device__ __attribute__((noinline)) inline V2<double> kernel_far64(const SysConst<double>& C, double t)
{
    V2<double> v;
    kernel_eval<double>(C, t, v.x, v.y);
    return v;
}
__device__ __attribute__((noinline)) inline V2<float> kernel_far32(const SysConst<float>& C, float t)
{
    V2<float> v;
    kernel_eval<float>(C, t, v.x, v.y);
    return v;
}

// The first octaves of a system's FP32 table in LDS: entry id (the bits of v
// >> TAB_SHIFT) below end at et + 32 id, the zero entry at end; pairs from
// end on read the whole table in HBM
struct TabHead {
    const char* et;
    uint32_t end;
    const TabE* all;
};
// a system's FP64 table in LDS, at that LDS address
struct TabLds64 {
    uint32_t at;
};
constexpr uint32_t tab_end(const char*) { return TAB_END; }
__device__ __forceinline__ uint32_t tab_end(const TabHead& h) { return h.end; }
__device__ __forceinline__ const char* tab_at(const char* et) { return et; }
__device__ __forceinline__ const char* tab_at(const TabHead& h) { return h.et; }
__device__ __forceinline__ bool tab64_at(const char* et, double t, double ts, double& Ht, double& H2)
{
    return tab64_lookup(et, t, ts, Ht, H2);
}
__device__ __forceinline__ bool tab64_at(const TabLds64& h, double t, double ts, double& Ht, double& H2)
{
    return tab64_lookup<true>(nullptr, t, ts, Ht, H2, h.at);
}

// copy the first octaves of one system's FP32 table (end - TAB_BIAS entries
// and a zero entry) from HBM into LDS
__device__ __forceinline__ void tab_load_head(const TabSys* g, TabE* tab, int entries, int tid, int nthreads)
{
    const float4* src = reinterpret_cast<const float4*>(g->e);
    float4* dst = reinterpret_cast<float4*>(tab);
    constexpr int EV = (int)(sizeof(TabE) / sizeof(float4));
    for (int i = tid; i < (entries + 1) * EV; i += nthreads)
        dst[i] = i < entries * EV ? src[i] : make_float4(0.f, 0.f, 0.f, 0.f);
}

// error-free (hi, lo) += d  (TwoSum, then renormalize)
template <typename T> __device__ __forceinline__ void acc2(T& hi, T& lo, T d)
{
    const T s = hi + d;
    const T bv = s - hi;
    const T e = (hi - (s - bv)) + (d - bv);
    const T l = lo + e;
    const T h = s + l;
    lo = l - (h - s);
    hi = h;
}

// ---------------------------------------------------------------------------
// symmetric pair schedule of the persistent kernel.  H1 and H2 depend on the
// pair distance only, and the contribution of a pair is even in d, so one
// evaluation serves both ends: target i gains Ht F_j + H2 (F_j . d) d and
// source j gains Ht F_i + H2 (F_i . d) d (eq. BrV).  Points form blocks of
// 64 (one per lane); for blocks a <= b, lane l pairs its point 64a + l with
// the point 64b + (l + s) mod 64 at offset s, s = 0..63 for a < b and
// s = 1..32 within a block (s = 32 pairs each couple twice, so lanes 32..63
// skip it).  The accumulator of the moving point rotates down one lane per
// offset.  All offsets of all block pairs (32 B^2 for B blocks) are split
// into WPS equal contiguous ranges, one per wave.  Each block is stored twice
// in a row (src2), so the point at offset s is read at lane + s.
// ---------------------------------------------------------------------------

// value of lane (l + 1) mod 64 (wave_rol:1; every lane has a source, so no
// fallback value is needed)
__device__ __forceinline__ float lane_rot(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x134, 0xF, 0xF, false));
}
__device__ __forceinline__ double lane_rot(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x134, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x134, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// v as an opaque wave-uniform value (a scalar register the compiler cannot
// fold into constants)
__device__ __forceinline__ int opaque_uniform(int v)
{
    int r;
    asm volatile("s_mov_b32 %0, %1" : "=s"(r) : "s"(v));
    return r;
}

// The base that pair_kernel reads a table by.  FP32: the entry of index id lies
// at et + (id << 5) bytes, so the bias goes into a wave-uniform base (a
// register operand of the address arithmetic; gfx9 address arithmetic takes no
// 32-bit literal).
template <typename T, int WRAP> __device__ __forceinline__ const char* tab_base(const void* tab)
{
    const char* et = reinterpret_cast<const char*>(tab);
    if constexpr (!WRAP && sizeof(T) == 4) et += opaque_uniform(-(int)(TAB_BIAS * sizeof(TabE)));
    return et;
}
template <typename T, int WRAP> __device__ __forceinline__ TabLds64 tab_base(TabLds64 tab) { return tab; }
template <typename T, int WRAP> __device__ __forceinline__ TabHead tab_base(TabHead tab)
{
    tab.et += opaque_uniform(-(int)(TAB_BIAS * sizeof(TabE)));
    return tab;
}

// slot of point i in the doubled source array
__device__ __forceinline__ int src2_slot(int i) { return ((i >> 6) << 7) + (i & 63); }

// the scheduler moves nothing over this point
__device__ __forceinline__ void reads_stay()
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// One pair's entry of the index window (at LDS address 0) on its way: the loads
// are issued where it is looked up, the kernel functions formed where they are
// needed
struct WinLook {
    uint32_t bits;
    TabE e;
    __device__ __forceinline__ void fetch(float dx, float dy)
    {
        bits = __builtin_bit_cast(uint32_t, fmaf(dx, dx, fmaf(dy, dy, 1.0f)));
#if defined(__HIP_DEVICE_COMPILE__)
        // (LDS addresses, which only the device pass compiles)
        struct alignas(16) Half {
            float c[4];
        };
        typedef const __attribute__((address_space(3))) Half* LdsHalf;
        const uint32_t at = tab_win_off(bits);
        const Half h = *(LdsHalf)(uintptr_t)at, g = *(LdsHalf)(uintptr_t)(at + TAB_WIN_G);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            e.h[k] = h.c[k];
            e.g[k] = g.c[k];
        }
#endif
    }
    __device__ __forceinline__ void values(float& Ht, float& H2) const { tab_eval(e, tab_u(bits), Ht, H2); }
};

// kernel functions of one pair at offset (dx, dy) (FP32: positions scaled by
// rho): the table (FAR = false; a pair beyond it gives zeros and, with CHECK,
// sets far), or the direct evaluation of pairs beyond the table only (FAR =
// true; zeros for the others).  H2 comes scaled to the coordinates (H2 / sigma
// in FP32).  et: FP32 the table in LDS (or its first octaves, a TabHead: FAR
// then reads the rest of the table in HBM), FP64 in HBM.
template <typename T, bool FAR, bool CHECK = true, int WRAP = 0, typename Tab>
__device__ __forceinline__ void pair_kernel(const SysConst<T>& C, const Tab& et, T dx, T dy, T& Ht, T& H2,
                                            bool& far)
{
    if constexpr (sizeof(T) == 8) {
        const T t = fma_t(dx, dx, dy * dy);
        if constexpr (!FAR) {
            bool f;
            if constexpr (WRAP == 4)
                f = tab64_lookup<true>(nullptr, t, C.ts, Ht, H2);
            else
                f = tab64_at(et, t, C.ts, Ht, H2);
            if constexpr (CHECK) far = far || f;
        } else {
            Ht = (T)0;
            H2 = (T)0;
            if (tab64_index(fma_t(t, C.ts, (T)1)) >= (uint32_t)TAB_N) {
                const V2<T> v = kernel_far64(C, t);
                Ht = v.x;
                H2 = v.y;
            }
        }
    } else {
        const uint32_t bits = __builtin_bit_cast(uint32_t, fmaf(dx, dx, fmaf(dy, dy, 1.0f)));
        const uint32_t id = bits >> TAB_SHIFT;
        if constexpr (!FAR) {
            if constexpr (CHECK) far = far || id >= tab_end(et);
            if constexpr (WRAP != 0) {
                WinLook e;
                e.fetch(dx, dy);
                e.values(Ht, H2);
            } else {
                tab_eval(*reinterpret_cast<const TabE*>(tab_at(et) + (min(id, tab_end(et)) << 5)), tab_u(bits), Ht, H2);
            }
        } else {
            Ht = 0.0f;
            H2 = 0.0f;
            if (id >= TAB_END) {
                const V2<float> v = kernel_far32(C, fmaf(dx, dx, dy * dy) * C.its);
                Ht = v.x;
                H2 = v.y * C.its;
            } else if constexpr (std::is_same<Tab, TabHead>::value) {
                if (id >= et.end) tab_eval(et.all[id - TAB_BIAS], tab_u(bits), Ht, H2);
            }
        }
    }
}

// offsets [s_lo, s_hi) of block pair (a, b); adds the target sums to block
// a's and the moving points' sums to block b's accumulators of this lane
template <typename T, int TPL, bool FAR, bool CHECK = true, int WRAP = 0, typename Tab>
__device__ __forceinline__ bool sym_offsets(const SysConst<T>& C, const Tab& et, const Src4<T>* src2, int a, int b,
                                            int s_lo, int s_hi, int lane, T (&accx)[TPL], T (&accy)[TPL])
{
    const Src4<T> ti = src2[(a << 7) + lane];
    const Src4<T>* sp = src2 + (b << 7) + lane;
    T ax = (T)0, ay = (T)0, bx = (T)0, by = (T)0;
    bool far = false;
    // offsets every lane takes (wave-uniform: a scalar loop counter), two
    // per iteration (one address update for both loads)
    const int s_full = __builtin_amdgcn_readfirstlane((a == b) ? min(s_hi, 32) : s_hi);
    // the pair's 2x2 tensor Ht I + H2 d d^T (5 operations) applied to both
    // ends' forces (8 FMAs): 13 operations against 14 for the two dot
    // products F.d, their scaling by H2 and the four terms of each end
    auto apply = [&](const Src4<T>& q, T dx, T dy, T Ht, T H2) {
        const T hx = H2 * dx, hy = H2 * dy;
        const T mxx = fma_t(hx, dx, Ht), myy = fma_t(hy, dy, Ht), mxy = hx * dy;
        ax = fma_t(mxx, q.fx, fma_t(mxy, q.fy, ax));
        ay = fma_t(mxy, q.fx, fma_t(myy, q.fy, ay));
        bx = lane_rot(fma_t(mxx, ti.fx, fma_t(mxy, ti.fy, bx)));
        by = lane_rot(fma_t(mxy, ti.fx, fma_t(myy, ti.fy, by)));
    };
    auto offset = [&](const Src4<T>& q) {
        const T dx = ti.x - q.x, dy = ti.y - q.y;
        T Ht, H2;
        pair_kernel<T, FAR, CHECK, WRAP>(C, et, dx, dy, Ht, H2, far);
        apply(q, dx, dy, Ht, H2);
    };
    int s = __builtin_amdgcn_readfirstlane(s_lo);
    if constexpr (WRAP == 2) {
        // one offset ahead with the table entry and two with the point, so that
        // neither LDS read is waited for where it is issued (the last ones lie
        // past the range, within the workgroup's LDS, and are dropped).  Pays
        // where a SIMD has two waves; its eight register moves do not where it
        // has four
        struct Stage {
            Src4<T> q;
            T dx, dy;
            WinLook e;
        };
        auto look = [&](Stage& g) {
            g.dx = ti.x - g.q.x;
            g.dy = ti.y - g.q.y;
            g.e.fetch(g.dx, g.dy);
        };
        // the stage's offset; its place goes to the next point
        auto take = [&](Stage& g, const Src4<T>& next) {
            T Ht, H2;
            g.e.values(Ht, H2);
            apply(g.q, g.dx, g.dy, Ht, H2);
            g.q = next;
        };
        if (s < s_full) {
            Stage g0, g1;
            g0.q = sp[s];
            g1.q = sp[s + 1];
            look(g0);
            for (; s + 1 < s_full; s += 2) {
                look(g1);
                const Src4<T> n0 = sp[s + 2];
                reads_stay();
                take(g0, n0);
                look(g0);
                const Src4<T> n1 = sp[s + 3];
                reads_stay();
                take(g1, n1);
            }
            if (s < s_full) take(g0, g0.q);
        }
    } else if constexpr (FAR) {
#pragma unroll 1
        for (; s < s_full; ++s) offset(sp[s]);
    } else {
        for (; s + 1 < s_full; s += 2) {
            offset(sp[s]);
            offset(sp[s + 1]);
        }
        if (s < s_full) offset(sp[s]);
    }
    if (s_full < s_hi) {
        // offset 32 within a block: lanes 32..63 repeat lanes 0..31's couples
        const Src4<T> q = sp[32];
        const T dx = ti.x - q.x, dy = ti.y - q.y;
        T Ht, H2;
        pair_kernel<T, FAR, CHECK, WRAP>(C, et, dx, dy, Ht, H2, far);
        Ht = lane < 32 ? Ht : (T)0;
        H2 = lane < 32 ? H2 : (T)0;
        const T hx = H2 * dx, hy = H2 * dy;
        const T mxx = fma_t(hx, dx, Ht), myy = fma_t(hy, dy, Ht), mxy = hx * dy;
        ax = fma_t(mxx, q.fx, fma_t(mxy, q.fy, ax));
        ay = fma_t(mxy, q.fx, fma_t(myy, q.fy, ay));
        bx = lane_rot(fma_t(mxx, ti.fx, fma_t(mxy, ti.fy, bx)));
        by = lane_rot(fma_t(mxy, ti.fx, fma_t(myy, ti.fy, by)));
    }
    // lane l now holds the sums of point (l + s_hi) mod 64 of block b
    const int from = (lane - s_hi) & 63;
    bx = __shfl(bx, from, 64);
    by = __shfl(by, from, 64);
#pragma unroll
    for (int c = 0; c < TPL; ++c) {
        if (c == a) {
            accx[c] += ax;
            accy[c] += ay;
        }
        if (c == b) {
            accx[c] += bx;
            accy[c] += by;
        }
    }
    return far;
}

// this wave's share of the pair sums of all n points: accx[c], accy[c] hold
// the partial velocity of point 64c + lane.  CHECK = false: the caller
// guarantees that no FP32 pair lies beyond the table, which then is read
// without the per-pair test (an index beyond it reads a zero entry).
// WRAP: the table at LDS address 0: 1: FP32, its index window (tab_load_window);
// 2: the same, read ahead; 4: FP64
template <typename T, int TPL, int WPS, bool CHECK = true, int WRAP = 0, typename Tab>
__device__ __forceinline__ void pair_phase_sym(const SysConst<T>& C, const Tab& tab, const Src4<T>* src2, int n,
                                               int wave, int lane, T (&accx)[TPL], T (&accy)[TPL])
{
#pragma unroll
    for (int c = 0; c < TPL; ++c) accx[c] = accy[c] = (T)0;
    const auto et = tab_base<T, WRAP>(tab);
    const int B = (n + 63) >> 6;
    const int S = 32 * B * B;
    const int per = (S + WPS - 1) / WPS;
    const int g0 = min(S, wave * per), g1 = min(S, g0 + per);
    int g = 0;  // first offset index of block pair (a, b)
    for (int a = 0; a < B && g < g1; ++a) {
        for (int b = a; b < B && g < g1; ++b) {
            const int len = (a == b) ? 32 : 64, base = (a == b) ? 1 : 0;
            const int lo = max(g0, g), hi = min(g1, g + len);
            if (lo < hi) {
                const int s_lo = lo - g + base, s_hi = hi - g + base;
                const bool far =
                    sym_offsets<T, TPL, false, CHECK, WRAP>(C, et, src2, a, b, s_lo, s_hi, lane, accx, accy);
                if constexpr (CHECK) {
                    if (__any(far)) sym_offsets<T, TPL, true>(C, et, src2, a, b, s_lo, s_hi, lane, accx, accy);
                }
            }
            g += len;
        }
    }
}

// The single block pair (a, b) and offset range [s_lo, s_hi) of this wave's
// share of pair_phase_sym's schedule for n points, when the share lies in
// one block pair (as for 128 points over 8 waves: 16 offsets each), else
// false.  Step-invariant: a run finds it once.
template <int WPS>
__device__ __forceinline__ bool sym_one_segment(int n, int wave, int& sa, int& sb, int& s_lo, int& s_hi)
{
    const int B = (n + 63) >> 6;
    const int S = 32 * B * B;
    const int per = (S + WPS - 1) / WPS;
    const int g0 = min(S, wave * per), g1 = min(S, g0 + per);
    if (g0 >= g1) return false;
    int g = 0;
    for (int a = 0; a < B; ++a) {
        for (int b = a; b < B; ++b) {
            const int len = (a == b) ? 32 : 64, base = (a == b) ? 1 : 0;
            if (g0 >= g && g1 <= g + len) {
                sa = a;
                sb = b;
                s_lo = g0 - g + base;
                s_hi = g1 - g + base;
                return true;
            }
            g += len;
        }
    }
    return false;
}

// pair_phase_sym for a wave whose share is the one segment found by
// sym_one_segment (same sums, same order)
template <typename T, int TPL, bool CHECK = true, int WRAP = 0, typename Tab>
__device__ __forceinline__ void pair_phase_seg(const SysConst<T>& C, const Tab& tab, const Src4<T>* src2, int a,
                                               int b, int s_lo, int s_hi, int lane, T (&accx)[TPL], T (&accy)[TPL])
{
#pragma unroll
    for (int c = 0; c < TPL; ++c) accx[c] = accy[c] = (T)0;
    const auto et = tab_base<T, WRAP>(tab);
    const bool far = sym_offsets<T, TPL, false, CHECK, WRAP>(C, et, src2, a, b, s_lo, s_hi, lane, accx, accy);
    if constexpr (CHECK) {
        if (__any(far)) sym_offsets<T, TPL, true>(C, et, src2, a, b, s_lo, s_hi, lane, accx, accy);
    }
}

// sum over the 64 lanes of a wavefront (butterfly; lane j's result is
// deterministic)
template <typename T> __device__ __forceinline__ T wave_total(T v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// v of the lane that lies R lanes further on (cyclically) in its row of 16
template <int R> __device__ __forceinline__ float row_rot(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 + R, 0xF, 0xF, false));
}
template <int R> __device__ __forceinline__ double row_rot(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + R, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + R, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// lanes 0..31: v.x + v.x of the lane 32 above; lanes 32..63: v.y + v.y of the
// lane 32 below (a swap of register halves, then one addition)
__device__ __forceinline__ float half_sums(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                    false, false);
    const uint32_t a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
// even rows of 16 lanes: x + x of the next row; odd rows: y + y of the row before
__device__ __forceinline__ float row_sums(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y),
                                                    false, false);
    const uint32_t a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ double half_sums(double x, double y)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, x), b = __builtin_bit_cast(uint64_t, y);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double row_sums(double x, double y)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, x), b = __builtin_bit_cast(uint64_t, y);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
// value of one lane in every lane
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double lane_value(double v, int l)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// One wave's share of the symmetric schedule of B blocks as where it starts
// (block pair (a, b), offset s) and how many offsets it takes: the shares of
// pair_phase_sym.  Step-invariant: a run finds it once.
struct PairShare {
    int a, b, s, count;
};
template <int WPS> __device__ __forceinline__ PairShare pair_share(int B, int wave)
{
    const int S = 32 * B * B, per = (S + WPS - 1) / WPS;
    const int g0 = min(S, wave * per);
    PairShare p{0, 0, 1, min(S, g0 + per) - g0};
    int g = g0;
    for (int len = 32; p.count > 0 && g >= len; len = p.a == p.b ? 32 : 64) {
        g -= len;
        if (++p.b == B) p.b = ++p.a;
    }
    p.s = g + (p.a == p.b ? 1 : 0);
    return p;
}

// the pair sums of one share (the sums of pair_phase_sym in its order, as one
// piece of code for any share)
template <typename T, int TPL, typename Tab>
__device__ __forceinline__ void pair_walk(const SysConst<T>& C, const Tab& tab, const Src4<T>* src2, int B,
                                          PairShare p, int lane, T (&accx)[TPL], T (&accy)[TPL])
{
#pragma unroll
    for (int c = 0; c < TPL; ++c) accx[c] = accy[c] = (T)0;
    const auto et = tab_base<T, false>(tab);
    while (p.count > 0) {
        const int hi = min(p.s + p.count, p.a == p.b ? 33 : 64);
        const bool far = sym_offsets<T, TPL, false>(C, et, src2, p.a, p.b, p.s, hi, lane, accx, accy);
        if (__any(far)) sym_offsets<T, TPL, true>(C, et, src2, p.a, p.b, p.s, hi, lane, accx, accy);
        p.count -= hi - p.s;
        if (++p.b == B) p.b = ++p.a;
        p.s = p.a == p.b ? 1 : 0;
    }
}

// Whether the tail schedule below does less work than the padded symmetric
// one for n points: r tail points (n = 64 Bf + r, 0 < r < 64) cost about
// r (33 Bf + 52) lane-operations per lane against 33 for each of the
// 32 (2 Bf + 1) offsets the padded last block adds.
__host__ __device__ constexpr bool tail_pays(int n)
{
    const int Bf = n >> 6, r = n & 63;
    return r != 0 && r * (33 * Bf + 52) < 33 * 32 * (2 * Bf + 1);
}

// Pair sums of n points whose last block is partly filled (r = n - 64 Bf
// points, 0 < r < 64): the symmetric schedule covers the Bf full blocks,
// and the r tail points take their pairs point by point instead of as a
// padded block of 64:
//  * tail point j against full block a: lane l evaluates the pair
//    (64 a + l, tail j) once; point 64 a + l keeps its share, and the
//    shares of tail point j, summed over all full blocks in each lane, are
//    summed over the wavefront once and kept by lane j;
//  * tail point j as a source within the tail: lanes l < r take the pair
//    (tail l, tail j) for target tail l only.
// Every ordered pair is taken once; tail point j goes to wave j mod WPS, and the
// full blocks' part is pair_walk's.  The kernel values within the tail are
// evaluated for four, two or one sources at once in groups of lanes (r <= 16,
// 32, 63) and handed to the lanes that sum them; the sums over the wavefront
// take two tail points at once in register halves and rows (10 operations for
// four sums, without LDS), instead of one source, and one sum of six LDS
// permutes, at a time.
template <typename T, int TPL, int WPS, typename Tab>
__device__ __forceinline__ void pair_tail(const SysConst<T>& C, const Tab& tab, const Src4<T>* src2, int n, int wave,
                                          int lane, T (&accx)[TPL], T (&accy)[TPL])
{
    const int Bf = n >> 6, r = n & 63;
    const auto et = tab_base<T, false>(tab);
    const Src4<T>* tail = src2 + src2_slot(64 * Bf);
    // tail point q's pairs with the full blocks; its own sums in bx, by
    auto against_blocks = [&](const Src4<T>& q, T& bx, T& by) {
        bool far = false;
        bx = by = (T)0;
        auto pass = [&](auto far_tag) {
            constexpr bool FAR = decltype(far_tag)::value;
#pragma unroll
            for (int a = 0; a < TPL; ++a) {
                if (a < Bf) {
                    const Src4<T> ti = src2[(a << 7) + lane];
                    const T dx = ti.x - q.x, dy = ti.y - q.y;
                    T Ht, H2;
                    pair_kernel<T, FAR>(C, et, dx, dy, Ht, H2, far);
                    const T hx = H2 * dx, hy = H2 * dy;
                    const T mxx = fma_t(hx, dx, Ht), myy = fma_t(hy, dy, Ht), mxy = hx * dy;
                    accx[a] = fma_t(mxx, q.fx, fma_t(mxy, q.fy, accx[a]));
                    accy[a] = fma_t(mxy, q.fx, fma_t(myy, q.fy, accy[a]));
                    bx = fma_t(mxx, ti.fx, fma_t(mxy, ti.fy, bx));
                    by = fma_t(mxy, ti.fx, fma_t(myy, ti.fy, by));
                }
            }
        };
        pass(std::integral_constant<bool, false>());
        if (__any(far)) pass(std::integral_constant<bool, true>());
    };
    const bool live = lane < r;
    const Src4<T> tp = tail[live ? lane : r - 1];
    const int lg = r <= 16 ? 4 : r <= 32 ? 5 : 6, L = 1 << lg;  // lanes of a group
    const Src4<T> gp = tail[min(lane & (L - 1), r - 1)];
    // kernel values of (tail point lane mod L, tail point j + WPS group)
    auto kernel_values = [&](int j, T& Ht, T& H2) {
        const Src4<T> q = tail[min(j + WPS * (lane >> lg), r - 1)];
        const T dx = gp.x - q.x, dy = gp.y - q.y;
        bool far = false;
        pair_kernel<T, false>(C, et, dx, dy, Ht, H2, far);
        if (__any(far)) {
            T Hf, Gf;
            pair_kernel<T, true>(C, et, dx, dy, Hf, Gf, far);
            Ht += Hf;  // one of the two is zero
            H2 += Gf;
        }
    };
    T tx = (T)0, ty = (T)0;  // sums of tail point `lane`
    T h = (T)0, g = (T)0, h2 = (T)0, g2 = (T)0;
    int at = 0;  // group of tail point j
    for (int j = wave; j < r; j += 2 * WPS) {
        const int j2 = j + WPS;
        if (at == 0) kernel_values(j, h, g);
        T hj = h, gj = g, hk, gk;
        if (lg == 6) {
            kernel_values(min(j2, r - 1), h2, g2);
            hk = h2;
            gk = g2;
        } else {
            const int from = (at << lg) + (lane & (L - 1));
            hj = __shfl(h, from, 64);
            gj = __shfl(g, from, 64);
            hk = __shfl(h, from + L, 64);
            gk = __shfl(g, from + L, 64);
            at = lg == 4 ? at ^ 2 : 0;
        }
        const Src4<T> q = tail[j], q2 = tail[min(j2, r - 1)];
        T bx = (T)0, by = (T)0, cx = (T)0, cy = (T)0;
        if (Bf > 0) {
            against_blocks(q, bx, by);
            if (j2 < r) against_blocks(q2, cx, cy);
        }
        // rows 0..3: x of j, x of j2, y of j, y of j2
        T z = row_sums(half_sums(bx, by), half_sums(cx, cy));
        z += row_rot<8>(z);
        z += row_rot<4>(z);
        z += row_rot<2>(z);
        z += row_rot<1>(z);
        auto within = [&](const Src4<T>& s, T Ht, T H2, int js, T sx, T sy) {
            const T dx = tp.x - s.x, dy = tp.y - s.y;
            Ht = live ? Ht : (T)0;
            H2 = live ? H2 : (T)0;
            const T fdj = H2 * fma_t(s.fx, dx, s.fy * dy);
            tx = fma_t(Ht, s.fx, fma_t(fdj, dx, tx));
            ty = fma_t(Ht, s.fy, fma_t(fdj, dy, ty));
            tx += lane == js ? sx : (T)0;
            ty += lane == js ? sy : (T)0;
        };
        within(q, hj, gj, j, lane_value(z, 0), lane_value(z, 32));
        if (j2 < r) within(q2, hk, gk, j2, lane_value(z, 16), lane_value(z, 48));
    }
#pragma unroll
    for (int c = 0; c < TPL; ++c) {
        if (c == Bf) {
            accx[c] += tx;
            accy[c] += ty;
        }
    }
}

}  // namespace swim
