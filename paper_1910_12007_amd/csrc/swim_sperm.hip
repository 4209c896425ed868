// swim_sperm.hip -- gfx950 forward run of the full sperm model of the
// Appendix: a flagellum with the tapered beat, a circular head (ring and
// diameter springs, head bending), the neck springs and the neck-angle
// energy, several swimmers per fluid, the dense regularized-Brinkmanlet sum
// of eq. (BrV) and the forward-Euler no-slip update (Sec. 2.1).
//
// One workgroup runs one system for all its steps (a persistent kernel fed
// by a work queue).  The pair sum uses the symmetric lane schedule of
// swim_pairsum.h, with the partly filled last block of 64 points taken
// point by point (74 points per swimmer leave 10 in it).  The elastic forces
// take two passes over the points: every point evaluates the curvature node it
// is the centre of and the spring to its next point (a head point its
// diameter, the first flagellum points the neck springs) into LDS, and after a
// barrier sums the terms it belongs to, in a fixed order without atomics.
//
// Discrete energy (trapezoid rule, centred differences; every spring has the
// form K (l/L0 - 1)^2 L0):
//   flagellum tension  K_T   segments k, k+1, rest ds
//   flagellum bending  K_C   (zeta_k - zhat_k)^2 ds at nodes 1..nf-2,
//                      zhat = d^2/ds^2 of a (1-s) sin(eta s - omega t + phase)
//   head ring          K_HT  neighbouring head points, rest the initial chord c
//   head diameters     K_HT  points pi apart, rest 2 H_r
//   head bending       K_HC  (kappa_m - 1/H_r)^2 c at every head node
//   neck springs       K_NT  last flagellum point to the head points at
//                      pi - dth, pi, pi + dth; the one before to pi -+ dth;
//                      rest the initial lengths
//   neck angle         K_NA  (z1 . z2)^2, z1 = H(pi) - F(nf-1),
//                      z2 = H(pi + dth) - H(pi - dth)
// F = -dE/dX (eq. Fenergy).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "swim.h"
#include "swim_internal.h"
#include "swim_math.h"
#include "swim_pairsum.h"

namespace swim {

namespace {

constexpr int32_t ST_BADPARAM = 3;

// positions of one point in LDS: FP32 (hi, lo) pairs, FP64 plain
template <typename T> struct PosE;
template <> struct alignas(16) PosE<float> {
    float xh, yh, xl, yl;
};
template <> struct alignas(16) PosE<double> {
    double xh, yh;
};

template <typename T> __device__ __forceinline__ PosE<T> pos_make(T xh, T yh, T xl, T yl)
{
    PosE<T> p;
    p.xh = xh;
    p.yh = yh;
    if constexpr (sizeof(T) == 4) {
        p.xl = xl;
        p.yl = yl;
    }
    return p;
}

// X_q - X_p (FP32: differences of the hi and of the lo parts)
template <typename T> __device__ __forceinline__ V2<T> pos_diff(const PosE<T>& q, const PosE<T>& p)
{
    V2<T> d;
    d.x = q.xh - p.xh;
    d.y = q.yh - p.yh;
    if constexpr (sizeof(T) == 4) {
        d.x += q.xl - p.xl;
        d.y += q.yl - p.yl;
    }
    return d;
}

// spring K (l/L0 - 1)^2 L0 between p and q: returns c with F_p += c (X_q - X_p),
// c = 2 K (l/L0 - 1)/l.  FP32 forms the strain as (l^2 - L0^2)/((l + L0) L0),
// free of the cancellation in l/L0 - 1.
template <typename T> __device__ __forceinline__ T spring_coef(V2<T> d, T L0, T L02, T K2)
{
    if constexpr (sizeof(T) == 4) {
        const float t2 = fmaf(d.x, d.x, d.y * d.y);
        const float rl = __builtin_amdgcn_rsqf(t2);
        const float l = t2 * rl;
        const float num = fmaf(d.x, d.x, fmaf(d.y, d.y, -L02));
        return K2 * num * __builtin_amdgcn_rcpf((l + L0) * L0) * rl;
    } else {
        const double l = sqrt(fma(d.x, d.x, d.y * d.y));
        return K2 * (l / L0 - 1.0) / l;
    }
}

// curvature node (A, B, C) with segments d1 = X_B - X_A, d2 = X_C - X_B and
// parameter step h: energy E = W (kappa - k0)^2 h; f[r] = dkappa/dX of the
// point in role r (0: A, 1: B, 2: C) of this node; returns dE/dkappa.
template <typename T>
__device__ __forceinline__ T node_terms(V2<T> d1, V2<T> d2, T inv2h, T invh2, T h, T W2, T k0, V2<T> (&f)[3])
{
    const T a = (d2.x + d1.x) * inv2h;
    const T b = (d2.y + d1.y) * inv2h;
    const T p = (d2.x - d1.x) * invh2;
    const T q = (d2.y - d1.y) * invh2;
    const T S = fma_t(a, a, b * b);
    T rS, rS32;  // 1/S, S^(-3/2)
    if constexpr (sizeof(T) == 4) {
        const float rs = __builtin_amdgcn_rsqf(S);
        rS = rs * rs;
        rS32 = rS * rs;
    } else {
        rS = 1.0 / S;
        rS32 = rS / sqrt(S);
    }
    const T num = fma_t(q, a, -p * b);
    const T co = W2 * (num * rS32 - k0) * h;  // dE/dkappa
    const T n3 = (T)3 * num * rS32 * rS;
    const T dka = q * rS32 - a * n3;
    const T dkb = -p * rS32 - b * n3;
    const T dkp = -b * rS32;
    const T dkq = a * rS32;
    // dkappa/dX of the point in role r
    f[0].x = fma_t(-dka, inv2h, dkp * invh2);
    f[0].y = fma_t(-dkb, inv2h, dkq * invh2);
    f[1].x = (T)-2 * dkp * invh2;
    f[1].y = (T)-2 * dkq * invh2;
    f[2].x = fma_t(dka, inv2h, dkp * invh2);
    f[2].y = fma_t(dkb, inv2h, dkq * invh2);
    return co;
}

// what one point evaluates and which terms it gathers (indices of the
// system's points; step-invariant).  Its chain is the flagellum or, closed to
// a ring, the head.
template <typename T> struct SpermPt {
    int pv, nx;      // neighbours in its chain (itself at the flagellum's ends)
    int ps;          // point whose next-spring is its previous one (the last flagellum point's, zero, for the first)
    int sa, sb;      // ends of its second spring: a diameter, or a neck spring
    int edge;        // the neck springs' slot it writes, or -1
    int role;        // 1..5: neck point nf-1, nf-2, c-1, c, c+1
    bool node, next, head;  // it is the centre of a curvature node, has a next-spring, lies in the head
    T inv2h, invh2, h, W2;  // node
    T L0, L02, K2;          // next-spring
    T M0, M02, J2;          // second spring
    T zA, zB;               // flagellum: preferred curvature zA cos(omega t) + zB sin(omega t)
};

// neck spring q (slot order: nf-1 to c-1, c, c+1; nf-2 to c-1, c+1)
__device__ __forceinline__ int neck_from(const SpermShape& g, int q) { return q < 3 ? g.nf - 1 : g.nf - 2; }
__device__ __forceinline__ int neck_to(const SpermShape& g, int q)
{
    const int c = g.nf + g.nh / 2;
    return q < 3 ? c - 1 + q : q == 3 ? c - 1 : c + 1;
}

// (cos x, sin x); not inlined: the argument reduction's registers and literals
// would stay allocated through the step loop (202 VGPRs, two waves per SIMD)
__device__ __attribute__((noinline)) V2<double> cos_sin(double x)
{
    V2<double> v;
    sincos(x, &v.y, &v.x);
    return v;
}

template <typename T>
__device__ SpermPt<T> sperm_point(const SpermShape& g, const double* sp, double phase, int base, int p)
{
    SpermPt<T> P;
    const int nf = g.nf, nh = g.nh, c = nf + nh / 2;
    P.head = p >= nf;
    P.edge = -1;
    P.zA = P.zB = (T)0;
    P.M0 = P.M02 = (T)1;
    P.J2 = (T)0;
    int pv, nx, ps, sa = p, sb = p;
    if (P.head) {
        const int m = p - nf;
        pv = nf + (m + nh - 1) % nh;
        nx = nf + (m + 1) % nh;
        ps = pv;
        sb = nf + (m + nh / 2) % nh;
        P.node = P.next = true;
        P.inv2h = (T)(0.5 / g.ch);
        P.invh2 = (T)(1.0 / (g.ch * g.ch));
        P.h = P.L0 = (T)g.ch;
        P.L02 = (T)(g.ch * g.ch);
        P.W2 = (T)(2.0 * sp[SWIM_SP_KHC]);
        P.K2 = P.J2 = (T)(2.0 * sp[SWIM_SP_KHT]);
        P.M0 = (T)(2.0 * g.hr);
        P.M02 = (T)(4.0 * g.hr * g.hr);
    } else {
        pv = max(p - 1, 0);
        nx = min(p + 1, nf - 1);
        ps = p >= 1 ? p - 1 : nf - 1;
        P.node = p >= 1 && p <= nf - 2;
        P.next = p <= nf - 2;
        P.inv2h = (T)(0.5 / g.ds);
        P.invh2 = (T)(1.0 / (g.ds * g.ds));
        P.h = P.L0 = (T)g.ds;
        P.L02 = (T)(g.ds * g.ds);
        P.W2 = (T)(2.0 * sp[SWIM_SP_KC]);
        P.K2 = (T)(2.0 * sp[SWIM_SP_KT]);
        if (p < 5) {
            P.edge = p;
            sa = neck_from(g, p);
            sb = neck_to(g, p);
            P.M0 = (T)g.L0[p];
            P.M02 = (T)(g.L0[p] * g.L0[p]);
            P.J2 = (T)(2.0 * sp[SWIM_SP_KNT]);
        }
        if (P.node) {
            const double a = sp[SWIM_SP_A], eta = sp[SWIM_SP_ETA];
            const double sj = (double)p * g.ds, psi = eta * sj + phase;
            const double u = -2.0 * a * eta, v = a * (1.0 - sj) * eta * eta;
            const V2<double> cs = cos_sin(psi);
            P.zA = (T)(u * cs.x - v * cs.y);
            P.zB = (T)(u * cs.y + v * cs.x);
        }
    }
    P.role = p == nf - 1 ? 1 : p == nf - 2 ? 2 : p == c - 1 ? 3 : p == c ? 4 : p == c + 1 ? 5 : 0;
    P.pv = base + pv;
    P.nx = base + nx;
    P.ps = base + ps;
    P.sa = base + sa;
    P.sb = base + sb;
    return P;
}

// the terms in LDS: per point the node's curvature gradients at its neighbours
// and the next-spring's force, per swimmer the neck springs
template <typename T> struct SpermTerms {
    Src4<T>* ends;  // [n] (f[0], f[2]) of the node
    Src4<T>* next;  // [n] (the next-spring's force, the node's dE/dkappa, unused)
    Src4<T>* neck;  // [5 nsw] (coefficient, d, unused)
};

// initial position of point p of a swimmer whose first flagellum point is (x0, y0)
__device__ __forceinline__ void sperm_initial(const SpermShape& g, double x0, double y0, int p, double& x, double& y)
{
    if (p < g.nf) {
        x = x0 + (double)p * g.ds;
        y = y0;
    } else {
        const int m = p - g.nf;
        const double xc = (x0 + (double)(g.nf - 1) * g.ds) + g.hr + g.dn;
        const V2<double> cs = cos_sin((double)m * g.dth);
        x = xc + g.hr * cs.x;
        y = y0 + g.hr * cs.y;
    }
}

struct SpermLdsLayout {
    size_t tab, src, part, pos, bad, total;
};
__host__ __device__ constexpr size_t al16(size_t x) { return (x + 15) & ~(size_t)15; }
// n points of nsw swimmers, the table's first oct octaves (FP64: all or none).
// The terms of
// the forces and the partial sums share one region: each is read before the
// barrier that the other is written behind.
__host__ __device__ constexpr SpermLdsLayout sperm_lds_layout(int dtype, int wps, int n, int nsw, int oct)
{
    const size_t e = dtype == 0 ? 4 : 8, nb = ((size_t)n + 63) / 64;
    const size_t part = (size_t)wps * n * 2 * e, terms = ((size_t)n * 8 + 20 * (size_t)nsw) * e;
    SpermLdsLayout L{};
    L.tab = 0;
    L.src = dtype == 0 ? ((size_t)(oct << TAB_M) + 1) * sizeof(TabE) : oct ? sizeof(TabSys64) : 0;
    L.part = al16(L.src + 128 * nb * 4 * e);
    L.pos = al16(L.part + (part > terms ? part : terms));
    L.bad = al16(L.pos + (size_t)n * 16);
    L.total = al16(L.bad + 4 * (size_t)wps);
    return L;
}

template <typename T> __device__ __forceinline__ Src4<T> neck_term(V2<T> d, T cf)
{
    Src4<T> v;
    v.x = cf;
    v.y = d.x;
    v.fx = d.y;
    v.fy = (T)0;
    return v;
}

// neck spring of rest length L0 from point p to point q (not inlined: only a
// flagellum of four points needs it apart)
template <typename T>
__device__ __attribute__((noinline)) void neck_spring(const PosE<T>* p, const PosE<T>* q, T L0, T L02, T K2,
                                                      Src4<T>* to)
{
    const V2<T> d = pos_diff(*q, *p);
    *to = neck_term(d, spring_coef(d, L0, L02, K2));
}

template <typename T, int TPL, int WPS, bool L64>
__device__ void sperm_system(const SpermShape& g, const SpermRun& r, int64_t s, const SysConst<T>& C,
                             const void* tab_g, TabE* tab_s, Src4<T>* src, V2<T>* part, PosE<T>* pos, int* badw,
                             T* head, T* tail, int32_t* status)
{
    constexpr bool COMP = sizeof(T) == 4;
    constexpr int NMAX = 64 * TPL, NT = 64 * WPS, PPT = (NMAX + NT - 1) / NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nf = g.nf, hc = g.nh / 2, np = nf + g.nh, nsw = g.nsw, n = np * nsw;
    const int nobs1 = r.n_obs + 1;
    const double* sp = r.sysp + (int64_t)SWIM_SP_NPARAM * s;
    const double* sw = r.swp + (int64_t)3 * nsw * s;
    T* hd = head + (int64_t)s * nsw * nobs1 * 2;
    T* tl = tail + (int64_t)s * nsw * nobs1 * 2;
    // samples a stopped (or not run) system does not reach stay NaN
    for (int k = tid; k < nsw * nobs1 * 2; k += NT) {
        hd[k] = (T)NAN;
        tl[k] = (T)NAN;
    }
    if (status[s] == ST_BADPARAM) {
        __syncthreads();
        return;
    }
    // FP32: the table's first octaves copied into LDS; FP64 reads it in place, or
    // (L64) copies all of it
    std::conditional_t<COMP, TabHead, std::conditional_t<L64, TabLds64, const void*>> tab;
    if constexpr (COMP) {
        const TabSys* all = (const TabSys*)tab_g + s;
        tab_load_head(all, tab_s, r.oct << TAB_M, tid, NT);
        tab = TabHead{reinterpret_cast<const char*>(tab_s), TAB_BIAS + ((uint32_t)r.oct << TAB_M), all->e};
    } else if constexpr (L64) {
        const float4* from = reinterpret_cast<const float4*>((const TabSys64*)tab_g + s);
#pragma unroll 4
        for (int i = tid; i < (int)(sizeof(TabSys64) / 16); i += NT) reinterpret_cast<float4*>(tab_s)[i] = from[i];
#if defined(__HIP_DEVICE_COMPILE__)
        tab = TabLds64{(uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)tab_s};
#endif
    } else {
        tab = (const TabSys64*)tab_g + s;
    }
    const T kna2 = (T)(2.0 * sp[SWIM_SP_KNA]), kh0 = (T)(1.0 / g.hr);
    const double om = sp[SWIM_SP_OMEGA];
    const T dt = (T)r.dt;
    const T rho = COMP ? C.tr : (T)1;

    // owned points i = tid + NT k: positions in registers
    T xh[PPT], yh[PPT], xl[PPT], yl[PPT];
    SpermPt<T> pt[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int i = tid + NT * k;
        const bool held = i < n;
        const int m = held ? i / np : 0, p = held ? i - m * np : 0;
        double X = 0.0, Y = 0.0;
        if (held) sperm_initial(g, sw[3 * m], sw[3 * m + 1], p, X, Y);
        xh[k] = (T)X;
        yh[k] = (T)Y;
        xl[k] = COMP ? (T)(X - (double)xh[k]) : (T)0;
        yl[k] = COMP ? (T)(Y - (double)yh[k]) : (T)0;
        if (held) pos[i] = pos_make<T>(xh[k], yh[k], xl[k], yl[k]);
        pt[k] = sperm_point<T>(g, sp, held ? sw[3 * m + 2] : 0.0, m * np, p);
        if (pt[k].edge >= 0) pt[k].edge += 5 * m;
    }
    // padding points n .. 64 B - 1 of the last block: no force, at the start
    // position of point n - 1 (they add nothing to the sums)
    for (int i = n + tid; i < 64 * ((n + 63) >> 6); i += NT) {
        double X, Y;
        sperm_initial(g, sw[3 * (nsw - 1)], sw[3 * (nsw - 1) + 1], np - 1, X, Y);
        Src4<T> v;
        v.x = (T)X * rho;
        v.y = (T)Y * rho;
        v.fx = (T)0;
        v.fy = (T)0;
        const int slot = src2_slot(i);
        src[slot] = v;
        src[slot + 64] = v;
    }
    // cos, sin of omega t: FP32 runs rotate by omega dt in FP64, FP64 runs
    // evaluate them directly
    double rc = 1.0, rs = 0.0;
    const V2<double> rot = cos_sin(om * r.dt);
    __syncthreads();

    SpermTerms<T> tm;
    tm.ends = reinterpret_cast<Src4<T>*>(part);
    tm.next = tm.ends + n;
    tm.neck = tm.next + n;
    // forces at the current positions (pos in LDS) into src.  A point's terms
    // in order: its previous and next spring, the nodes next, own and previous,
    // a diameter, the neck.  (One pass in which every point evaluates each
    // spring and node it belongs to takes three nodes instead of one, in two
    // divergent halves for flagellum and head, and five neck branches.)
    auto forces = [&]() {
        V2<T> d2[PPT], f1[PPT], dm[PPT];
        T c2[PPT], cm[PPT], co[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int i = tid + NT * k;
            if (i < n) {
                const SpermPt<T>& P = pt[k];
                const PosE<T> X = pos_make<T>(xh[k], yh[k], xl[k], yl[k]);
                const V2<T> d1 = pos_diff(X, pos[P.pv]);
                d2[k] = pos_diff(pos[P.nx], X);
                const T zh = P.head ? kh0 : fma_t(P.zA, (T)rc, P.zB * (T)rs);
                V2<T> f[3];
                co[k] = node_terms<T>(d1, d2[k], P.inv2h, P.invh2, P.h, P.W2, zh, f);
                co[k] = P.node ? co[k] : (T)0;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    f[q].x = P.node ? f[q].x : (T)0;
                    f[q].y = P.node ? f[q].y : (T)0;
                }
                f1[k] = f[1];
                c2[k] = spring_coef(d2[k], P.L0, P.L02, P.K2);
                c2[k] = P.next ? c2[k] : (T)0;
                Src4<T> e;
                e.x = f[0].x;
                e.y = f[0].y;
                e.fx = f[2].x;
                e.fy = f[2].y;
                tm.ends[i] = e;
                Src4<T> sv;
                sv.x = c2[k] * d2[k].x;
                sv.y = c2[k] * d2[k].y;
                sv.fx = co[k];
                sv.fy = (T)0;
                tm.next[i] = sv;
                dm[k] = pos_diff(pos[P.sb], pos[P.sa]);
                cm[k] = spring_coef(dm[k], P.M0, P.M02, P.J2);
                if (P.edge >= 0) tm.neck[P.edge] = neck_term(dm[k], cm[k]);
                cm[k] = P.head ? cm[k] : (T)0;
                // (four flagellum points: the last takes neck spring 4, too)
                if (nf < 5 && P.role == 1)
                    neck_spring(pos + (i - 1), pos + (i + 2 + hc), (T)g.L0[4], (T)(g.L0[4] * g.L0[4]),
                                (T)(2.0 * sp[SWIM_SP_KNT]), tm.neck + 5 * ((i - 3) / np) + 4);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int i = tid + NT * k;
            if (i < n) {
                const SpermPt<T>& P = pt[k];
                const Src4<T> sp0 = tm.next[P.ps];
                const Src4<T> en = tm.ends[P.nx], ep = tm.ends[P.pv];
                const T con = tm.next[P.nx].fx, cop = tm.next[P.pv].fx;
                V2<T> F;
                F.x = fma_t(c2[k], d2[k].x, -sp0.x);
                F.y = fma_t(c2[k], d2[k].y, -sp0.y);
                F.x = fma_t(-cop, ep.fx, fma_t(-co[k], f1[k].x, fma_t(-con, en.x, F.x)));
                F.y = fma_t(-cop, ep.fy, fma_t(-co[k], f1[k].y, fma_t(-con, en.y, F.y)));
                F.x = fma_t(cm[k], dm[k].x, F.x);
                F.y = fma_t(cm[k], dm[k].y, F.y);
                if (P.role != 0) {
                    // the neck springs this point ends, then the neck angle:
                    // E = K (z1.z2)^2, dE/dz1 = 2K (z1.z2) z2, dE/dz2 = 2K (z1.z2) z1
                    const int base = P.role == 1 ? i - (nf - 1) : P.role == 2 ? i - (nf - 2) : i - (nf + hc) - (P.role - 4);
                    const Src4<T>* N = tm.neck + 5 * (base / np);
                    const T sg = P.role <= 2 ? (T)1 : (T)-1;
                    auto add = [&](int q) {
                        const Src4<T> e = N[q];
                        F.x = fma_t(e.x, sg * e.y, F.x);
                        F.y = fma_t(e.x, sg * e.fx, F.y);
                    };
                    if (P.role == 1 || P.role == 3) add(0);
                    if (P.role == 2 || P.role == 3) add(3);
                    if (P.role == 1 || P.role == 4) add(1);
                    if (P.role == 1 || P.role == 5) add(2);
                    if (P.role == 2 || P.role == 5) add(4);
                    if (P.role != 2) {
                        const int c = base + nf + hc;
                        V2<T> z1;
                        z1.x = N[1].y;
                        z1.y = N[1].fx;
                        const V2<T> z2 = pos_diff(pos[c + 1], pos[c - 1]);
                        const T w = kna2 * fma_t(z1.x, z2.x, z1.y * z2.y);
                        const V2<T> z = (P.role == 1 || P.role == 4) ? z2 : z1;
                        const T sw = (P.role == 1 || P.role == 3) ? w : -w;
                        F.x = fma_t(sw, z.x, F.x);
                        F.y = fma_t(sw, z.y, F.y);
                    }
                }
                Src4<T> v;
                v.x = xh[k] * rho;
                v.y = yh[k] * rho;
                v.fx = F.x;
                v.fy = F.y;
                const int slot = src2_slot(i);
                src[slot] = v;
                src[slot + 64] = v;
            }
        }
    };
    auto observe = [&](int o) {
        for (int m = tid; m < nsw; m += NT) {
            double cx = 0.0, cy = 0.0;
            const PosE<T>* P = pos + m * np;
            for (int j = g.nf; j < np; ++j) {
                cx += (double)P[j].xh;
                cy += (double)P[j].yh;
                if constexpr (COMP) {
                    cx += (double)P[j].xl;
                    cy += (double)P[j].yl;
                }
            }
            T* h = hd + ((int64_t)m * nobs1 + o) * 2;
            T* t = tl + ((int64_t)m * nobs1 + o) * 2;
            h[0] = (T)(cx / (double)g.nh);
            h[1] = (T)(cy / (double)g.nh);
            double tx = (double)P[0].xh, ty = (double)P[0].yh;
            if constexpr (COMP) {
                tx += (double)P[0].xl;
                ty += (double)P[0].yl;
            }
            t[0] = (T)tx;
            t[1] = (T)ty;
        }
    };
    int st = 0;
    int obs_left = r.obs_every, obs_k = 0;
    bool due = true;  // an observation of the present positions
    // this wave's share of the symmetric schedule (of the full blocks when
    // the tail schedule takes the rest)
    const bool tail_sched = tail_pays(n);
    const int B = tail_sched ? n >> 6 : (n + 63) >> 6;
    PairShare share = pair_share<WPS>(B, wave);
    share.a = __builtin_amdgcn_readfirstlane(share.a);
    share.b = __builtin_amdgcn_readfirstlane(share.b);
    share.s = __builtin_amdgcn_readfirstlane(share.s);
    share.count = __builtin_amdgcn_readfirstlane(share.count);
    for (int step = 0;; ++step) {
        if (due) observe(obs_k++);
        if (step == r.steps) break;
        forces();
        __syncthreads();
        {
            T ax[TPL], ay[TPL];
            pair_walk<T, TPL>(C, tab, src, B, share, lane, ax, ay);
            if (tail_sched) pair_tail<T, TPL, WPS>(C, tab, src, n, wave, lane, ax, ay);
#pragma unroll
            for (int c = 0; c < TPL; ++c) {
                if (64 * c + lane < n) {
                    V2<T> v;
                    v.x = ax[c];
                    v.y = ay[c];
                    part[wave * n + 64 * c + lane] = v;
                }
            }
        }
        __syncthreads();
        // Euler step of the owned points; partial sums reduced in wave order
        int bad = 0;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int i = tid + NT * k;
            if (i < n) {
                V2<T> pv[WPS];
#pragma unroll
                for (int w = 0; w < WPS; ++w) pv[w] = part[w * n + i];
                T ux = (T)0, uy = (T)0;
#pragma unroll
                for (int w = 0; w < WPS; ++w) {
                    ux += pv[w].x;
                    uy += pv[w].y;
                }
                if constexpr (COMP) {
                    acc2(xh[k], xl[k], dt * ux);
                    acc2(yh[k], yl[k], dt * uy);
                } else {
                    xh[k] = fma_t(dt, ux, xh[k]);
                    yh[k] = fma_t(dt, uy, yh[k]);
                }
                if (bad_t(xh[k]) || bad_t(yh[k])) bad = max(bad, (isfinite(xh[k]) && isfinite(yh[k])) ? 2 : 1);
                pos[i] = pos_make<T>(xh[k], yh[k], xl[k], yl[k]);
            }
        }
        if constexpr (COMP) {
            const double c0 = rc;
            rc = fma(c0, rot.x, -rs * rot.y);
            rs = fma(rs, rot.x, c0 * rot.y);
        } else {
            const V2<double> cs = cos_sin(om * ((double)(step + 1) * r.dt));
            rc = cs.x;
            rs = cs.y;
        }
        {
            const bool b1 = __ballot(bad == 1) != 0, b2 = __ballot(bad == 2) != 0;
            if (lane == 0) badw[wave] = (b1 ? 1 : 0) | (b2 ? 2 : 0);
        }
        __syncthreads();
        const int bw = lane < WPS ? badw[lane] : 0;
        const int bflags = (__ballot(bw & 1) ? 1 : 0) | (__ballot(bw & 2) ? 2 : 0);
        if (bflags) {
            st = (bflags & 1) ? 1 : 2;
            break;
        }
        due = r.obs_every > 0 && --obs_left == 0;
        if (due) obs_left = r.obs_every;
    }
    if (tid == 0) status[s] = st;
    __syncthreads();
}

// Bound by VALU issue in large batches (about 2300 wave-operations a step of 74
// points, 1350 of them the pairs'), by the chain of one step in small ones.
// Large batches therefore want the waves that hide a step's four barriers and
// table reads: 128 VGPRs (the far-field evaluation and the trigonometry called,
// not inlined; 25..34 step-invariant values spilled to scratch) and 20 KB of LDS
// (24 octaves of the table) let eight systems of two waves share a CU, where 202
// VGPRs allowed four.  With the forces in two
// passes and the tail sums in registers, 2000 one-swimmer systems take 8.2 us
// per step against 14.7, 1024 5.6 against 7.8, one system 3.3 against 4.6; 1000
// of two swimmers 15.7 against 19.1 (above 128 points 128 VGPRs spill more, and 168
// measure 18.8).
// L64: FP64 with the table in LDS, for launches whose workgroups share no CU
// (from the caches a pair's nine 16-byte reads are bound by the L1): one system
// 10.5 -> 7.2 us per step, four of two swimmers 27 -> 12.6.
template <typename T, int TPL, int WPS, bool L64 = false>
__global__ __launch_bounds__(64 * WPS, sizeof(T) == 4 && TPL <= 2 ? 4 : 1) void k_sperm_forward(
    SpermShape g, SpermRun r, const SysConst<T>* sysc, const void* tabs, int32_t* queue, T* head, T* tail,
    int32_t* status)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_item;
    const SpermLdsLayout lay =
        sperm_lds_layout(sizeof(T) == 4 ? 0 : 1, WPS, g.nsw * (g.nf + g.nh), g.nsw, r.oct);
    TabE* tab = reinterpret_cast<TabE*>(smem + lay.tab);
    Src4<T>* src = reinterpret_cast<Src4<T>*>(smem + lay.src);
    V2<T>* part = reinterpret_cast<V2<T>*>(smem + lay.part);
    PosE<T>* pos = reinterpret_cast<PosE<T>*>(smem + lay.pos);
    int* badw = reinterpret_cast<int*>(smem + lay.bad);
    // work queue: a workgroup takes at most n_sys items, so the loop ends
    for (int64_t it = 0; it <= r.n_sys; ++it) {
        if (threadIdx.x == 0) s_item = atomicAdd(queue, 1);
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        if (item >= r.n_sys) break;
        sperm_system<T, TPL, WPS, L64>(g, r, item, sysc[item], tabs, tab, src, part, pos, badw, head, tail, status);
    }
}

// per-system constants, one wave per system; rows outside the model's domain
// are flagged
template <typename T>
__global__ __launch_bounds__(64) void k_sperm_setup(int32_t nsw, double eps, const double* sysp, const double* swp,
                                                    SysConst<T>* sysc, SysConst<double>* sysc64, int32_t* status,
                                                    int blob)
{
    const int64_t s = blockIdx.x;
    const int lane = threadIdx.x;
    const double* p = sysp + (int64_t)SWIM_SP_NPARAM * s;
    const double alpha = p[SWIM_SP_ALPHA];
    bool ok = isfinite(alpha) && alpha >= 0.0 && alpha * eps <= 1.0;
    for (int c = lane; c < SWIM_SP_NPARAM; c += 64) ok = ok && isfinite(p[c]);
    for (int c = lane; c < 3 * nsw; c += 64) ok = ok && isfinite(swp[(int64_t)3 * nsw * s + c]);
    ok = __all(ok);
    if (lane == 0) status[s] = ok ? 0 : ST_BADPARAM;
    sysconst_wave<T>(ok ? alpha : 0.0, eps, sysc + s, sysc64 ? sysc64 + s : nullptr, blob, lane);
}

// observables of a sperm run per system s and interval/sample k = 1..n_obs
// (Sec. 4): kind 0, the head-centre velocity of swimmer 0,
// (h_k - h_{k-1}) / dt_obs; kind 1, the distance between the tail ends and
// between the head centres of swimmers 0 and 1 at sample k.  Stopped runs
// give NaN.
template <typename T>
__global__ void k_sperm_observables(int kind, int64_t n_sys, int32_t nsw, int32_t n_obs, double dt_obs, const T* head,
                                    const T* tail, const int32_t* status, double* g)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_sys * n_obs) return;
    const int64_t s = e / n_obs;
    const int k = (int)(e - s * n_obs) + 1;
    double* o = g + 2 * e;
    if (status[s] != 0) {
        o[0] = NAN;
        o[1] = NAN;
        return;
    }
    const int64_t stride = (int64_t)(n_obs + 1) * 2;  // one swimmer's samples
    const T* h0 = head + s * nsw * stride;
    if (kind == 0) {
        o[0] = ((double)h0[2 * k] - (double)h0[2 * k - 2]) / dt_obs;
        o[1] = ((double)h0[2 * k + 1] - (double)h0[2 * k - 1]) / dt_obs;
    } else {
        const T* t0 = tail + s * nsw * stride;
        const T *h1 = h0 + stride, *t1 = t0 + stride;
        const double tx = (double)t0[2 * k] - (double)t1[2 * k], ty = (double)t0[2 * k + 1] - (double)t1[2 * k + 1];
        const double hx = (double)h0[2 * k] - (double)h1[2 * k], hy = (double)h0[2 * k + 1] - (double)h1[2 * k + 1];
        o[0] = sqrt(fma(tx, tx, ty * ty));
        o[1] = sqrt(fma(hx, hx, hy * hy));
    }
}

// Gaussian log-likelihood (eqs. likelihood, fitness) with a diagonal
// covariance of two levels: entries 0, 2, 4, ... (the odd entries in 1-based
// numbering) have standard deviation sig2[2i], the others sig2[2i+1].
// A stopped run or a non-finite output gives -inf.
__global__ void k_gauss_loglik2(int64_t n, int32_t n_obs, const double* g, const double* data, const double* sig2,
                                const int32_t* status, double* logl)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double* gi = g + i * (int64_t)n_obs * 2;
    double Ja = 0.0, Jb = 0.0;
    bool ok = status == nullptr || status[i] == 0;
    for (int k = 0; k < n_obs && ok; ++k) {
        ok = isfinite(gi[2 * k]) && isfinite(gi[2 * k + 1]);
        const double ra = data[2 * k] - gi[2 * k], rb = data[2 * k + 1] - gi[2 * k + 1];
        Ja = fma(ra, ra, Ja);
        Jb = fma(rb, rb, Jb);
    }
    if (!ok) {
        logl[i] = -INFINITY;
        return;
    }
    const double sa = sig2[2 * i], sb = sig2[2 * i + 1], m = (double)n_obs;
    if (!(sa > 0.0 && sb > 0.0)) {
        logl[i] = -INFINITY;
        return;
    }
    logl[i] = -m * log(2.0 * M_PI) - m * (log(sa) + log(sb)) - 0.5 * (Ja / (sa * sa) + Jb / (sb * sb));
}

size_t sperm_lds_bytes(int dtype, int wps, const SpermShape& g, int oct)
{
    return sperm_lds_layout(dtype, wps, g.nsw * (g.nf + g.nh), g.nsw, oct).total;
}

template <typename T, int TPL, int WPS>
hipError_t launch_sperm_t(int nblocks, const SpermShape& g, const SpermRun& r, const void* sysc, const void* tabs,
                          int32_t* queue, void* head, void* tail, int32_t* status, hipStream_t st)
{
    const size_t lds = sperm_lds_bytes(sizeof(T) == 4 ? 0 : 1, WPS, g, r.oct);
    if constexpr (sperm_lds64(sizeof(T) == 4 ? 0 : 1, TPL, WPS)) {
        if (r.oct) {
            hipLaunchKernelGGL((k_sperm_forward<T, TPL, WPS, true>), dim3(nblocks), dim3(64 * WPS), lds, st, g, r,
                               (const SysConst<T>*)sysc, tabs, queue, (T*)head, (T*)tail, status);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_sperm_forward<T, TPL, WPS>), dim3(nblocks), dim3(64 * WPS), lds, st, g, r,
                       (const SysConst<T>*)sysc, tabs, queue, (T*)head, (T*)tail, status);
    return hipGetLastError();
}

template <typename T, int TPL, int WPS> const void* sperm_kernel_ptr()
{
    return reinterpret_cast<const void*>(&k_sperm_forward<T, TPL, WPS>);
}

// dispatch over (dtype, tpl, wps); f receives the instantiation's tag types
template <typename F> hipError_t sperm_dispatch(int dtype, int tpl, int wps, F f)
{
#define SWIM_SPERM_CASE(TT, TP, WP)                                      \
    if (tpl == TP && wps == WP) return f((TT*)nullptr, std::integral_constant<int, TP>(), \
                                         std::integral_constant<int, WP>());
#define SWIM_SPERM_WPS(TT, TP) SWIM_SPERM_CASE(TT, TP, 2) SWIM_SPERM_CASE(TT, TP, 4) SWIM_SPERM_CASE(TT, TP, 8)
#define SWIM_SPERM_ALL(TT) \
    SWIM_SPERM_WPS(TT, 1) SWIM_SPERM_WPS(TT, 2) SWIM_SPERM_WPS(TT, 3) SWIM_SPERM_WPS(TT, 4) SWIM_SPERM_WPS(TT, 6) \
    SWIM_SPERM_WPS(TT, 8)
    if (dtype == 0) {
        SWIM_SPERM_ALL(float)
    } else {
        SWIM_SPERM_ALL(double)
    }
#undef SWIM_SPERM_ALL
#undef SWIM_SPERM_WPS
#undef SWIM_SPERM_CASE
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_sperm_setup(int dtype, int64_t n_sys, int32_t nsw, double eps, const double* sysp,
                              const double* swp, void* sysc, void* sysc64, int32_t* status, int blob,
                              hipStream_t st)
{
    if (n_sys == 0) return hipSuccess;
    if (!grid_fits(n_sys, 64)) return hipErrorInvalidConfiguration;
    const unsigned nb = (unsigned)n_sys;
    if (dtype == 0)
        hipLaunchKernelGGL(k_sperm_setup<float>, dim3(nb), dim3(64), 0, st, nsw, eps, sysp, swp,
                           (SysConst<float>*)sysc, (SysConst<double>*)sysc64, status, blob);
    else
        hipLaunchKernelGGL(k_sperm_setup<double>, dim3(nb), dim3(64), 0, st, nsw, eps, sysp, swp,
                           (SysConst<double>*)sysc, (SysConst<double>*)nullptr, status, blob);
    return hipGetLastError();
}

hipError_t prepare_sperm(int dtype, int tpl, int wps)
{
    return sperm_dispatch(dtype, tpl, wps, [&](auto* tt, auto tp, auto wp) {
        using T = std::remove_pointer_t<decltype(tt)>;
        const void* k = sperm_kernel_ptr<T, decltype(tp)::value, decltype(wp)::value>();
        // (the most that any call of this instantiation takes: a call must not
        // lower the limit that another thread's launch needs)
        const size_t most = sperm_lds_layout(dtype, wps, 64 * tpl, 8 * tpl, dtype == 0 ? TAB_OCT : 0).total;
        if constexpr (sperm_lds64(sizeof(T) == 4 ? 0 : 1, decltype(tp)::value, decltype(wp)::value)) {
            const void* k64 =
                reinterpret_cast<const void*>(&k_sperm_forward<T, decltype(tp)::value, decltype(wp)::value, true>);
            const hipError_t e = hipFuncSetAttribute(k64, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)sperm_lds_layout(1, wps, 64 * tpl, 8 * tpl, 1).total);
            if (e != hipSuccess) return e;
        }
        return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
    });
}

int sperm_blocks_per_cu(int dtype, int tpl, int wps, const SpermShape& g, int oct)
{
    int nb = 0;
    const hipError_t e = sperm_dispatch(dtype, tpl, wps, [&](auto* tt, auto tp, auto wp) {
        using T = std::remove_pointer_t<decltype(tt)>;
        const void* k = sperm_kernel_ptr<T, decltype(tp)::value, decltype(wp)::value>();
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, 64 * wps, sperm_lds_bytes(dtype, wps, g, oct));
    });
    return (e == hipSuccess && nb > 0) ? nb : 1;
}

hipError_t launch_sperm_forward(int dtype, int tpl, int wps, int nblocks, const SpermShape& g, const SpermRun& r,
                                const void* sysc, const void* tabs, int32_t* queue, void* head, void* tail,
                                int32_t* status, hipStream_t st)
{
    return sperm_dispatch(dtype, tpl, wps, [&](auto* tt, auto tp, auto wp) {
        using T = std::remove_pointer_t<decltype(tt)>;
        return launch_sperm_t<T, decltype(tp)::value, decltype(wp)::value>(nblocks, g, r, sysc, tabs, queue, head,
                                                                           tail, status, st);
    });
}

hipError_t launch_sperm_observables(int dtype, int kind, int64_t n_sys, int32_t nsw, int32_t n_obs, double dt_obs,
                                    const void* head, const void* tail, const int32_t* status, double* g,
                                    hipStream_t st)
{
    const int64_t m = n_sys * n_obs;
    if (m == 0) return hipSuccess;
    const unsigned nb = (unsigned)((m + 255) / 256);
    if (dtype == 0)
        hipLaunchKernelGGL(k_sperm_observables<float>, dim3(nb), dim3(256), 0, st, kind, n_sys, nsw, n_obs, dt_obs,
                           (const float*)head, (const float*)tail, status, g);
    else
        hipLaunchKernelGGL(k_sperm_observables<double>, dim3(nb), dim3(256), 0, st, kind, n_sys, nsw, n_obs, dt_obs,
                           (const double*)head, (const double*)tail, status, g);
    return hipGetLastError();
}

hipError_t launch_gauss_loglik2(int64_t n, int32_t n_obs, const double* g, const double* data, const double* sig2,
                                const int32_t* status, double* logl, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gauss_loglik2, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, n_obs, g, data, sig2,
                       status, logl);
    return hipGetLastError();
}

}  // namespace swim
