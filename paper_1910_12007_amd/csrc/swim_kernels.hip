// swim_kernels.hip -- gfx950 kernels of the batched filament-swimmer forward
// model (Sec. 2.1 and the Appendix): preferred curvature and elastic forces
// (eqs. EFB, curva, EFT, Fenergy), the dense regularized-Brinkmanlet velocity
// sum (eq. BrV), the forward-Euler no-slip update, head observations, and the
// ABC distance / tolerance kernels around it.
//
// Precision: every kernel is one template instantiated for float and double.
// In float the filament positions are carried as (hi, lo) pairs updated by an
// error-free TwoSum, so the segment vectors that drive the stiff stretching
// springs keep full relative precision.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "swim_internal.h"
#include "swim_math.h"
#include "swim_pairsum.h"

namespace swim {

constexpr int32_t SWIM_ST_BADPARAM_ = 3;
constexpr int32_t SWIM_ST_REJECTED_ = 4;


// LDS ordering between lanes of one wavefront: a wavefront's LDS operations
// execute in issue order, so a compiler-level fence around a wave barrier is
// enough to order a store by one lane before a later load by another.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T> __device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ float sin_t(float x) { return sinf(x); }
__device__ __forceinline__ double sin_t(double x) { return sin(x); }

// parameters of one filament, in the working precision
template <typename T> struct FilP {
    T Sb, Ss, b, om, kw, ph, ds, inv2ds, invds2;
    int N;
};

template <typename T>
__device__ __forceinline__ FilP<T> load_filp(const double* params, int64_t f, int N)
{
    const double* P = params + 9 * f;
    FilP<T> q;
    q.Sb = (T)P[1];
    q.Ss = (T)P[2];
    q.b = (T)P[3];
    q.om = (T)P[4];
    q.kw = (T)P[5];
    q.ph = (T)P[6];
    const double ds = 1.0 / (double)(N - 1);
    q.ds = (T)ds;
    q.inv2ds = (T)(0.5 / ds);
    q.invds2 = (T)(1.0 / (ds * ds));
    q.N = N;
    return q;
}

// Force F_p = -dE/dX_p on point p of one filament from the discrete tensile
// energy S_s sum_k (l_k/ds - 1)^2 ds and bending energy
// S_b sum_{k=1}^{N-2} (kappa_k - kappa0_k)^2 ds (Appendix EFT, EFB, curva;
// centred differences, interior nodes only).  seg(k, dx, dy) returns the
// segment vector X_{k+1} - X_k.
template <typename T, typename Seg>
__device__ __forceinline__ void point_force(const Seg& seg, int p, const FilP<T>& q, T t, T& Fx, T& Fy)
{
    const int N = q.N;
    T dx[4], dy[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int k = p - 2 + c;
        if (k >= 0 && k <= N - 2) {
            seg(k, dx[c], dy[c]);
        } else {
            dx[c] = (T)0;
            dy[c] = (T)0;
        }
    }
    Fx = (T)0;
    Fy = (T)0;
    // stretching: +tau_p (segment p) - tau_{p-1} (segment p-1)
#pragma unroll
    for (int c = 1; c <= 2; ++c) {
        const int k = p - 2 + c;
        if (k >= 0 && k <= N - 2) {
            const T l = sqrt_t(fma_t(dx[c], dx[c], dy[c] * dy[c]));
            const T co = (T)2 * q.Ss * (l / q.ds - (T)1) / l;
            const T sg = (c == 2) ? (T)1 : (T)-1;
            Fx = fma_t(sg * co, dx[c], Fx);
            Fy = fma_t(sg * co, dy[c], Fy);
        }
    }
    // bending: curvature nodes k = p-1, p, p+1
#pragma unroll
    for (int kk = -1; kk <= 1; ++kk) {
        const int k = p + kk;
        if (k < 1 || k > N - 2) continue;
        const int ca = kk + 1, cb = kk + 2;  // d_{k-1}, d_k
        const T a = (dx[cb] + dx[ca]) * q.inv2ds;
        const T bb = (dy[cb] + dy[ca]) * q.inv2ds;
        const T pp = (dx[cb] - dx[ca]) * q.invds2;
        const T qq = (dy[cb] - dy[ca]) * q.invds2;
        const T S = fma_t(a, a, bb * bb);
        const T rS = (T)1 / S;
        const T rS32 = rS / sqrt_t(S);
        const T num = fma_t(qq, a, -pp * bb);
        const T kap = num * rS32;
        const T k0 = -q.kw * q.kw * q.b * sin_t(fma_t(q.kw * q.ds, (T)k, q.ph - q.om * t));
        const T co = (T)2 * q.Sb * (kap - k0) * q.ds;
        const T n3 = (T)3 * num * rS32 * rS;
        const T dka = qq * rS32 - a * n3;
        const T dkb = -pp * rS32 - bb * n3;
        const T dkp = -bb * rS32;
        const T dkq = a * rS32;
        T gx, gy;
        if (kk == 1) {          // p = k - 1
            gx = fma_t(-dka, q.inv2ds, dkp * q.invds2);
            gy = fma_t(-dkb, q.inv2ds, dkq * q.invds2);
        } else if (kk == 0) {   // p = k
            gx = (T)-2 * dkp * q.invds2;
            gy = (T)-2 * dkq * q.invds2;
        } else {                // p = k + 1
            gx = fma_t(dka, q.inv2ds, dkp * q.invds2);
            gy = fma_t(dkb, q.inv2ds, dkq * q.invds2);
        }
        Fx = fma_t(-co, gx, Fx);
        Fy = fma_t(-co, gy, Fy);
    }
}

// Accumulate the velocity sum of eq. (BrV) over sources src[0..n) for the
// TPL targets (xi, yi) of this lane, with H1 taken relative to H1(0), in
// FP64 (FP32 lanes use pair_accumulate_x): kernel values from the system's
// FP64 table, pairs beyond it by direct evaluation in a second pass.  The
// constant part H1(0) sum_j F_j is the caller's: the velocity kernel for
// given forces adds it once per target; in a forward run the forces are the
// elastic forces of a translation-invariant energy (Appendix EFT, EFB), whose
// sum over the points of a filament is identically zero, so the term is zero
// and is not evaluated (its floating-point value is only rounding noise of
// the cancelling forces).
template <typename T, int TPL>
__device__ __forceinline__ void pair_accumulate(const SysConst<T>& C, const TabSys64* tab, const Src4<T>* src, int n,
                                                const T (&xi)[TPL], const T (&yi)[TPL],
                                                T (&ax)[TPL], T (&ay)[TPL])
{
    static_assert(sizeof(T) == 8, "FP64 only");
    auto add = [&](const Src4<T>& s, int k, T dx, T dy, T Ht, T H2) {
        const T h2fd = H2 * fma_t(s.fx, dx, s.fy * dy);
        ax[k] = fma_t(Ht, s.fx, fma_t(h2fd, dx, ax[k]));
        ay[k] = fma_t(Ht, s.fy, fma_t(h2fd, dy, ay[k]));
    };
    bool far = false;
    for (int j = 0; j < n; ++j) {
        const Src4<T> s = src[j];
#pragma unroll
        for (int k = 0; k < TPL; ++k) {
            const T dx = xi[k] - s.x, dy = yi[k] - s.y;
            T Ht, H2;
            far = tab64_lookup(tab, fma_t(dx, dx, dy * dy), C.ts, Ht, H2) || far;
            add(s, k, dx, dy, Ht, H2);
        }
    }
    if (__any(far)) {
        for (int j = 0; j < n; ++j) {
            const Src4<T> s = src[j];
#pragma unroll
            for (int k = 0; k < TPL; ++k) {
                const T dx = xi[k] - s.x, dy = yi[k] - s.y;
                const T t = fma_t(dx, dx, dy * dy);
                if (tab64_index(fma_t(t, C.ts, (T)1)) >= (uint32_t)TAB_N) {
                    const V2<T> v = kernel_far64(C, t);
                    add(s, k, dx, dy, v.x, v.y);
                }
            }
        }
    }
}

// FP32 pair sum with FP64 accumulation, for lanes that sum whole large
// systems.  Filament forces alternate in sign with magnitudes far above the
// velocity they produce (bending forces ~4e2 against velocities ~10 for
// N = 512), so the FP32 rounding of Ht * F_j (Ht ~ 0.3) and of an FP32
// running sum each leave ~1e-5 of relative error over thousands of sources.
// Here Ht = h0 + (h0lo + increment) keeps the constant term in two floats,
// the small in-interval increment is evaluated in FP32, and the products
// (exact in FP64) accumulate in FP64, which this chip issues at the FP32
// rate.  The H2 term stays in FP32 up to its product.
template <int TPL>
__device__ __forceinline__ void pair_accumulate_x(const SysConst<float>& C, const TabSys* tab,
                                                  const Src4<float>* src, int n, const float (&xi)[TPL],
                                                  const float (&yi)[TPL], double (&ax)[TPL], double (&ay)[TPL])
{
    uint32_t far = 0;
    const float ts = C.ts;
    for (int j = 0; j < n; ++j) {
        const Src4<float> s = src[j];
        const double fx = s.fx, fy = s.fy;
#pragma unroll
        for (int k = 0; k < TPL; ++k) {
            const float dx = xi[k] - s.x, dy = yi[k] - s.y;
            const uint32_t bits = tab_bits(fmaf(dx, dx, dy * dy), ts);
            const uint32_t id = bits >> TAB_SHIFT;
            far |= id >= TAB_END ? 1u : 0u;
            const uint32_t ic = min(id, TAB_END) - TAB_BIAS;
            const TabE& e = tab->e[ic];
            const float u = tab_u(bits);
            const float inc = u * fmaf(fmaf(e.h[3], u, e.h[2]), u, e.h[1]);
            const float lo = tab->h0lo[ic] + inc;
            const float H2 = fmaf(fmaf(fmaf(e.g[3], u, e.g[2]), u, e.g[1]), u, e.g[0]) * ts;
            const float h2fd = H2 * fmaf(s.fx, dx, s.fy * dy);
            ax[k] = fma((double)e.h[0], fx, fma((double)lo, fx, fma((double)h2fd, (double)dx, ax[k])));
            ay[k] = fma((double)e.h[0], fy, fma((double)lo, fy, fma((double)h2fd, (double)dy, ay[k])));
        }
    }
    if (__any(far)) {
        for (int j = 0; j < n; ++j) {
            const Src4<float> s = src[j];
#pragma unroll
            for (int k = 0; k < TPL; ++k) {
                const float dx = xi[k] - s.x, dy = yi[k] - s.y;
                const float t = fmaf(dx, dx, dy * dy);
                if ((tab_bits(t, ts) >> TAB_SHIFT) >= TAB_END) {
                    float Ht, H2;
                    kernel_eval<float>(C, t, Ht, H2);
                    const float h2fd = H2 * fmaf(s.fx, dx, s.fy * dy);
                    ax[k] = fma((double)Ht, (double)s.fx, fma((double)h2fd, (double)dx, ax[k]));
                    ay[k] = fma((double)Ht, (double)s.fy, fma((double)h2fd, (double)dy, ay[k]));
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// set-up
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(64) void k_sysconst(const double* alpha, const double* eps, SysConst<T>* out,
                                                 SysConst<double>* out64, int blob)
{
    const int64_t i = blockIdx.x;  // one wave per system
    sysconst_wave<T>(alpha[i], eps[i], out + i, out64 ? out64 + i : nullptr, blob, threadIdx.x);
}

// per-system constants of a forward batch; systems whose parameters leave
// the kernel's domain (alpha < 0, alpha*eps > 1, non-finite rows) are
// flagged SWIM_ST_BADPARAM_ and skipped by the run kernels.
template <typename T>
__global__ __launch_bounds__(64) void k_sysconst_batch(const int64_t* sw_off, const int32_t* npt, const double* params,
                                                       double eps_over_ds, SysConst<T>* out, SysConst<double>* out64,
                                                       int32_t* status, int blob)
{
    const int64_t s = blockIdx.x;  // one wave per system
    const int lane = threadIdx.x;
    const double alpha = params[9 * sw_off[s]];
    const double eps = eps_over_ds / (double)(npt[s] - 1);
    bool ok = isfinite(alpha) && alpha >= 0.0 && alpha * eps <= 1.0;
    for (int64_t k = 9 * sw_off[s] + lane; k < 9 * sw_off[s + 1]; k += 64) ok = ok && isfinite(params[k]);
    ok = __all(ok);
    if (lane == 0) status[s] = ok ? 0 : SWIM_ST_BADPARAM_;
    sysconst_wave<T>(ok ? alpha : 0.0, eps, out + s, out64 ? out64 + s : nullptr, blob, lane);
}

// FP32 kernel tables of systems [s0, s0 + n), one thread per interval; the
// FP64 evaluation's registers stay out of the kernels that use the tables
// One wave per TAB_CHUNK = 21 consecutive intervals of one system, one FP64
// kernel value per lane: lanes 3j, 3j + 1, 3j + 2 evaluate the nodes 0, 1/4,
// 3/4 of interval j, lane 63 the end of interval 20 (the next chunk's first
// node); lane 3j gathers the interval's four values (its node 1 is the next
// interval's node 0, at exactly the same t) and writes the entry.  Three
// kernel values per entry, each on its own lane.
constexpr int TAB_CHUNK = 21;
constexpr int TAB_WAVES = (TAB_N + 1 + TAB_CHUNK - 1) / TAB_CHUNK;  // waves per system

__global__ __launch_bounds__(64) void k_table_build(int64_t s0, int64_t n, const SysConst<double>* sysc64, TabSys* tab)
{
    const int64_t w = blockIdx.x;
    const int lane = threadIdx.x;
    const int64_t s = s0 + w / TAB_WAVES;
    const int j = lane < 3 * TAB_CHUNK ? lane / 3 : TAB_CHUNK, k = lane < 3 * TAB_CHUNK ? lane % 3 : 0;
    const int i = (int)(w % TAB_WAVES) * TAB_CHUNK + j;  // interval, or the end node (lane 63)
    const bool live = w < n * TAB_WAVES && i <= TAB_N && (k == 0 || i < TAB_N);
    double fh = 0.0, fg = 0.0;
    if (live) tab_node(sysc64[s], i, k, fh, fg);
    // every lane of the wave takes part in the shuffles
    double h[4], g[4];
    h[0] = fh;
    g[0] = fg;
#pragma unroll
    for (int d = 1; d < 4; ++d) {
        const int src = min(lane + d, 63);
        h[d] = __shfl(fh, src);
        g[d] = __shfl(fg, src);
    }
    if (!live || k != 0 || lane >= 3 * TAB_CHUNK) return;
    if (i == TAB_N) {
        tab_interval(sysc64[s], i, tab[s].e[i], &tab[s].h0lo[i]);  // the zero entry
        return;
    }
    TabE e;
    tab_assemble(sysc64[s], h, g, e, &tab[s].h0lo[i]);
    tab[s].e[i] = e;
}

// FP64 velocity sums: systems without a table (k_direct_velocity).  A table takes
// 6336 evaluations and 99 KB, the pairs of a few points less: 10000 systems of 10
// points at alpha = 0 88 us a call against 850, of 24 137 against 908; one system
// of 24 points, the reading's blob, 34 against 36, where the chain of its pairs
// catches up with the table's set-up.  By the system's own size, so that its bits do
// not depend on the call.
__device__ __forceinline__ bool direct64(const SysConst<double>& C, int64_t n)
{
    return C.paper != 2.0 && n <= DIRECT64_MAX;
}

// Kernel tables by the interval sweep (pb_iv_*), one workgroup of TAB_N
// threads per system, one interval per thread: FP32 tables with the paper's
// blob (K = 7 nodes), and FP64 tables of any blob (K = 9).  A system at
// alpha > 0 with the paper's blob (paper == 2):
//  1. each thread evaluates the Bessel functions at its interval's nodes
//     and totals the integrands of A and B;
//  2. exclusive prefix sums of A and suffix sums of B over the intervals;
//  3. the flux G at the nodes, totals of the integrands of g - g(0) and I2,
//     and their prefix sums;
//  4. the node values; intervals outside the sweep take the near-contact
//     series or the far field.
// Other systems evaluate their closed forms at the nodes.  Bound by the FP64
// Bessel functions (one set per node, ~250 operations); with one quadrature
// rule per gap between nodes instead (three 6-point rules per interval, a
// Bessel set at every point) 4096 FP32 tables took 1.2 ms and one 60 us.
constexpr int PB_BLOCK = TAB_N;
static_assert(PB_BLOCK % 64 == 0 && PB_BLOCK <= 1024, "one interval per thread");

// exclusive scans over the workgroup in thread order: a forward, b forward
// or (REVB) from the last thread down; red holds 2 PB_BLOCK / 64 values
template <bool REVB> __device__ void pb_block_scan2(double& a, double& b, double* red)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NW = PB_BLOCK / 64;
    const int l = REVB ? 63 - lane : lane;
    double ia = a, ib = b;  // inclusive within the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double ua = __shfl(ia, max(lane - o, 0), 64);
        const double ub = __shfl(ib, REVB ? min(lane + o, 63) : max(lane - o, 0), 64);
        if (lane >= o) ia += ua;
        if (l >= o) ib += ub;
    }
    __syncthreads();  // the previous scan's totals are read
    if (lane == 63) red[wave] = ia;
    if (l == 63) red[NW + wave] = ib;
    __syncthreads();
    double ba = 0.0, bb = 0.0;
    for (int w = 0; w < NW; ++w) {
        if (w < wave) ba += red[w];
        const int ww = REVB ? NW - 1 - w : w;
        if (REVB ? ww > wave : ww < wave) bb += red[NW + ww];
    }
    a = ba + ia - a;
    b = bb + ib - b;
}

template <int K>
__global__ __launch_bounds__(PB_BLOCK) void k_table_build_pb(int64_t s0, const SysConst<double>* __restrict__ sysc64,
                                                             void* __restrict__ tab, const int64_t* pt_off)
{
    __shared__ double s_red[2 * PB_BLOCK / 64];
    __shared__ double s_sh[PB_NSER - 1], s_sg[PB_NSER - 1];
    const int i = threadIdx.x;  // the interval
    const int64_t s = s0 + blockIdx.x;
    // read in place (uniform loads), not copied into per-lane registers
    const SysConst<double>& C = sysc64[s];
    if (pt_off && direct64(C, pt_off[s + 1] - pt_off[s])) return;
    const bool sweep = C.paper == 2.0;
    double fh[K], fg[K];
    int iS = TAB_N;
    if (sweep) {  // uniform over the workgroup
        const PbRange R = pb_range(C);
        iS = R.iS;
        const double alpha = sqrt(C.a2);
        const bool in = i >= R.iS && i < R.iE;
        double fa[K], fb[K], p[K], q[K];
        double A = 0.0, B = 0.0;
        if (i == TAB_N - 1) pb_series(C, s_sh, s_sg);
        if (in) {
            pb_iv_nodes<K, true>(C, alpha, i, fa, fb, p, q);
            A = lob_total<K>(fa);
            B = lob_total<K>(fb);
        } else if (i < R.iS) {
            pb_iv_nodes<K, false>(C, alpha, i, fa, fb, p, q);
            A = lob_total<K>(fa);
        }
        pb_block_scan2<true>(A, B, s_red);
        const bool own = in && i < R.iF;
        double D = 0.0, I2 = 0.0;
        if (own) {
            pb_iv_flux<K>(C, i, A, B, fa, fb, p, q);
            D = lob_total<K>(fa);
            I2 = lob_total<K>(fb);
        }
        pb_block_scan2<false>(D, I2, s_red);
        if (own) {
            // start values of the sweep from the series
            double v0, hv, h0, g0;
            tab_span(R.iS, v0, hv);
            const double t0 = (v0 - 1.0) * C.its;
            pb_series_eval(s_sh, s_sg, t0 * C.inv_e2, h0, g0);
            pb_iv_values<K>(C, i, D + (-2.0 * h0 - t0 * g0), I2 + t0 * (t0 * g0), fa, fb, fh, fg);
        } else {
            pb_iv_outside<K>(C, i, true, iS, s_sh, s_sg, fh, fg);
        }
    } else {
        pb_iv_outside<K>(C, i, false, iS, s_sh, s_sg, fh, fg);
    }
    if constexpr (K == 7) {
        TabSys& T = reinterpret_cast<TabSys*>(tab)[s];
        const double h4[4] = {fh[0], fh[2], fh[4], fh[6]}, g4[4] = {fg[0], fg[2], fg[4], fg[6]};
        TabE e;
        tab_assemble(C, h4, g4, e, &T.h0lo[i]);
        T.e[i] = e;
        if (i == 0) tab_interval(C, TAB_N, T.e[TAB_N], &T.h0lo[TAB_N]);  // the zero entry
    } else {
        tab64_entry(i, fh, fg, reinterpret_cast<TabSys64*>(tab)[s].e[i]);
    }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// the item of a prefix array (first[0..n], ascending) that index i falls in
__device__ __forceinline__ int64_t prefix_item(const int64_t* first, int64_t n, int64_t i)
{
    int64_t lo = 0, hi = n;  // first[lo] <= i < first[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) / 2;
        if (first[mid] <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// standalone dense velocity sum (one evaluation of eq. BrV), one-sided: a
// workgroup takes 64 targets of one system, one per lane, and its eight waves
// split the sources (streamed through LDS in tiles of 512) between them;
// the waves' sums are added in order.  blk0[s]: first workgroup of system s.
// Bound by the chain of pair evaluations per lane: with one wave per 64
// targets over all sources, 256 or 512 targets a workgroup, two FP64 systems
// of 200 points took 78 us.
// ---------------------------------------------------------------------------
constexpr int VEL_WAVES = 8, VEL_TILE = 512;
template <typename T>
__global__ __launch_bounds__(64 * VEL_WAVES) void k_pair_velocity(int64_t n_sys, const int64_t* blk0,
                                                                  const int64_t* pt_off, const SysConst<T>* sysc,
                                                                  const void* tabs, const T* x, const T* y,
                                                                  const T* fx, const T* fy, T* ux, T* uy)
{
    __shared__ Src4<T> tile[VEL_TILE];
    __shared__ V2<double> part[VEL_WAVES][64];
    __shared__ double red[2][VEL_WAVES];
    // the FP32 table (FP64 reads its own from HBM)
    __shared__ std::conditional_t<sizeof(T) == 4, TabSys, int> tab_s[1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t s = prefix_item(blk0, n_sys, blockIdx.x);
    const int64_t p0 = pt_off[s];
    const int64_t n = pt_off[s + 1] - p0;
    const int64_t i = ((int64_t)blockIdx.x - blk0[s]) * 64 + lane;
    const SysConst<T>& C = sysc[s];
    if constexpr (sizeof(T) == 4) tab_load((const TabSys*)tabs + s, tab_s, tid, 64 * VEL_WAVES);
    // FP32 accumulates in FP64 (pair_accumulate_x); FP64 in FP64
    const T xi[1] = {i < n ? x[p0 + i] : (T)0}, yi[1] = {i < n ? y[p0 + i] : (T)0};
    double ax[1] = {0.0}, ay[1] = {0.0};
    // sum of the forces in FP64: it multiplies H1(0) in every target's
    // velocity, and the forces of a filament cancel to a small total
    double sfx = 0.0, sfy = 0.0;
    for (int64_t j0 = 0; j0 < n; j0 += VEL_TILE) {
        const int64_t j = j0 + tid;
        Src4<T> v;
        if (j < n) {
            v.x = x[p0 + j];
            v.y = y[p0 + j];
            v.fx = fx[p0 + j];
            v.fy = fy[p0 + j];
            sfx += v.fx;
            sfy += v.fy;
        } else {
            v.x = v.y = v.fx = v.fy = (T)0;
        }
        __syncthreads();
        tile[tid] = v;
        __syncthreads();
        const int m = (int)min<int64_t>(VEL_TILE, n - j0), per = (m + VEL_WAVES - 1) / VEL_WAVES;
        const int lo = min(m, w * per), hi = min(m, lo + per);
        if constexpr (sizeof(T) == 4)
            pair_accumulate_x<1>(C, tab_s, tile + lo, hi - lo, xi, yi, ax, ay);
        else
            pair_accumulate<T, 1>(C, (const TabSys64*)tabs + s, tile + lo, hi - lo, xi, yi, ax, ay);
    }
    sfx = wave_sum(sfx);
    sfy = wave_sum(sfy);
    if (lane == 0) {
        red[0][w] = sfx;
        red[1][w] = sfy;
    }
    part[w][lane] = V2<double>{ax[0], ay[0]};
    __syncthreads();
    if (w != 0 || i >= n) return;
    double SFx = 0.0, SFy = 0.0, u = 0.0, v = 0.0;
#pragma unroll
    for (int k = 0; k < VEL_WAVES; ++k) {
        SFx += red[0][k];
        SFy += red[1][k];
        u += part[k][lane].x;
        v += part[k][lane].y;
    }
    ux[p0 + i] = (T)fma((double)C.h1c, SFx, u);
    uy[p0 + i] = (T)fma((double)C.h1c, SFy, v);
}

// FP64 systems of at most DIRECT64_MAX points with closed forms (direct64), a wave
// each: a target per lane, all sources in LDS.  blk0 as for the other sums.
__global__ __launch_bounds__(64) void k_direct_velocity(int64_t n_sys, const int64_t* blk0, const int64_t* pt_off,
                                                        const SysConst<double>* sysc, const double* x, const double* y,
                                                        const double* fx, const double* fy, double* ux, double* uy)
{
    __shared__ Src4<double> src[DIRECT64_MAX];
    const int lane = threadIdx.x;
    const int64_t s = prefix_item(blk0, n_sys, blockIdx.x);
    const int64_t p0 = pt_off[s];
    const int n = (int)(pt_off[s + 1] - p0);
    const SysConst<double>& C = sysc[s];
    Src4<double> own{};
    if (lane < n) src[lane] = own = Src4<double>{x[p0 + lane], y[p0 + lane], fx[p0 + lane], fy[p0 + lane]};
    __syncthreads();
    double u = 0.0, v = 0.0, sfx = 0.0, sfy = 0.0;
    for (int j = 0; j < n; ++j) {
        const Src4<double> q = src[j];
        const double dx = own.x - q.x, dy = own.y - q.y;
        double Ht, H2;
        kernel_eval_closed<double>(C, fma(dx, dx, dy * dy), Ht, H2);
        const double h2fd = H2 * fma(q.fx, dx, q.fy * dy);
        u = fma(Ht, q.fx, fma(h2fd, dx, u));
        v = fma(Ht, q.fy, fma(h2fd, dy, v));
        sfx += q.fx;
        sfy += q.fy;
    }
    if (lane < n) {
        ux[p0 + lane] = fma(C.h1c, sfx, u);
        uy[p0 + lane] = fma(C.h1c, sfy, v);
    }
}

// ---------------------------------------------------------------------------
// standalone elastic forces at time t (one thread per point)
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_forces(int64_t n_fil, const int64_t* fil_off, const int32_t* npt, const double* params,
                         double t, const T* x, const T* y, T* fx, T* fy)
{
    const int64_t f = blockIdx.y;
    if (f >= n_fil) return;
    const int N = npt[f];
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int64_t b = fil_off[f];
    const FilP<T> q = load_filp<T>(params, f, N);
    auto seg = [&](int k, T& dx, T& dy) {
        dx = x[b + k + 1] - x[b + k];
        dy = y[b + k + 1] - y[b + k];
    };
    T Fx, Fy;
    point_force<T>(seg, p, q, (T)t, Fx, Fy);
    fx[b + p] = Fx;
    fy[b + p] = Fy;
}


// FP32 launch shapes whose table is held as the 64 KiB LDS index window (an
// address without a bias and a clamp, two operations less per pair): those that
// run at most two systems per CU (eight waves up to 128 points) or one (16 waves
// above) anyway, where the windows and the rest of the layout fit the LDS
__host__ __device__ constexpr bool fwd_window(int dtype, int tpl, int wps)
{
    return dtype == 0 && ((tpl <= 2 && wps == 8) || (tpl >= 3 && wps == 16));
}

// Queue order of a merged bucket's systems when they outnumber its workgroups:
// the runs likely to go the whole way first, each group in the order given
// (largest first).  A launch lasts as long as its last long run.  Largest first
// alone ends with the smallest systems, but where most draws blow up within a
// few hundred steps the few long runs, small ones, start last (a generation of
// 16384 draws: 0.25 s against 0.20 with the smaller systems first); smaller
// first ends with the largest where all complete (1024 systems of 64..512 points,
// 500 steps: 31.4 ms, with this order 26.8; the draws' generations, 0.11..0.12 and
// 0.18..0.24 s from run to run, stay within that).  The forecast is forward Euler's bound on the bending
// modes, dt rho < 2 with rho = 5.5e4 (S_b / 0.1) (127 ds)^-3 (the paper's blob
// at eps = 1.5 ds; a margin of 10 %): it decides the order of independent runs,
// nothing else.  One workgroup per bucket, 4 us.
__global__ __launch_bounds__(1024) void k_order_runs(OrderSegs seg, const int32_t* in, const int64_t* sw_off,
                                                     const int32_t* npt, const double* params, double dt, int32_t* out)
{
    __shared__ uint64_t mask[ORDER_MAX / 64];
    __shared__ int32_t wtot[16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t i0 = seg.start[blockIdx.x];
    const int n = seg.count[blockIdx.x];
    int own = 0;  // long runs in this wave's words of the mask
    for (int k = tid; k < ((n + 63) & ~63); k += 1024) {
        bool longrun = false;
        if (k < n) {
            const int32_t s = in[i0 + k];
            const double r = 127.0 / (double)(npt[s] - 1);
            longrun = dt * 5.5e5 * params[9 * sw_off[s] + 1] < 2.2 * r * r * r;
        }
        const uint64_t m = __ballot(longrun);
        if (lane == 0) mask[k >> 6] = m;
        own += __popcll(m);
    }
    if (lane == 0) wtot[w] = own;
    __syncthreads();
    int total = 0;
    for (int k = 0; k < 16; ++k) total += wtot[k];
    // each wave takes a contiguous range of words, its offset the long runs
    // of the words before
    const int words = (n + 63) >> 6, per = (words + 15) / 16, w0 = min(words, w * per), w1 = min(words, w0 + per);
    int before = 0;
    for (int k = lane; k < w0; k += 64) before += __popcll(mask[k]);
    before = (int)wave_sum((float)before);
    for (int k = w0; k < w1; ++k) {
        const uint64_t m = mask[k];
        const int i = 64 * k + lane;
        if (i < n) {
            const int rank = before + __popcll(m & ((1ull << lane) - 1));  // long runs ahead of i
            out[i0 + ((m >> lane) & 1 ? rank : total + (i - rank))] = in[i0 + i];
        }
        before += __popcll(m);
    }
}

// LDS of the persistent kernel: [FP32 table][src2][part][bad, item], 16-byte
// aligned sections.  The kernel has no static LDS, so the table (or its
// index window) starts at LDS address 0 and a pair's entry address needs
// no base
struct FwdLdsLayout {
    size_t tab, src, part, bad, trig, total;
};
__host__ __device__ constexpr size_t fwd_align16(size_t x) { return (x + 15) & ~(size_t)15; }
// FP64 launch shapes that have a second build with the table in LDS (99 KB of
// it, so one workgroup per CU, as the registers of eight waves allow anyway: 214..246
// of 512 a lane).  Every launch of these shapes takes it from FWD_LDS64_STEPS steps
// on, however many systems or other launches there are: from the caches, a pair's
// nine 16-byte reads are bound by the L1's 64 bytes a clock.  2 runs of 64 points
// 3.4 -> 2.5 us a step, 4 of 200 points 36 -> 18, 300 of 200 points 8 steps 602
// -> 396 us; the copy is under 2 us per system, so runs of a few steps keep the
// caches.
__host__ __device__ constexpr bool fwd_lds64(int dtype, int tpl, int wps) { return dtype == 1 && tpl <= 4 && wps == 8; }
constexpr int FWD_LDS64_STEPS = 8;
__host__ __device__ constexpr FwdLdsLayout fwd_lds_layout(int dtype, int tpl, int wps, bool lds64 = false)
{
    const size_t e = dtype == 0 ? sizeof(float) : sizeof(double), nmax = 64 * (size_t)tpl;
    FwdLdsLayout L{};
    L.tab = 0;
    L.src = dtype == 0 ? fwd_align16(fwd_window(dtype, tpl, wps) ? TAB_WIN_BYTES : sizeof(TabSys))
            : lds64    ? sizeof(TabSys64)
                       : 0;
    L.part = fwd_align16(L.src + 2 * nmax * 4 * e);
    L.bad = fwd_align16(L.part + (size_t)wps * nmax * 2 * e);
    L.trig = fwd_align16(L.bad + 4 * ((size_t)wps + 1));  // (after the wave flags and the queue item)
    L.total = L.trig + (dtype == 0 ? 0 : 2 * (nmax / 3) * 16);
    return L;
}

// ---------------------------------------------------------------------------
// persistent forward run: one workgroup of WPS wavefronts per system, systems
// taken from a longest-first work queue; every time step stays inside the
// workgroup.  A step has two phases separated by barriers:
//
//  * pair phase (all waves): each wavefront sums over 1/WPS of the sources
//    (positions and forces in LDS; FP32 positions scaled by the table's rho)
//    for all targets and leaves its partial velocities in LDS;
//  * point phase (the first few waves): each wave covers a window of 60
//    consecutive points plus two halo points on either side, one point per
//    lane, with the positions kept in registers.  Lanes reduce the partial
//    velocities of their point in a fixed order (deterministic), take the
//    Euler step, and evaluate the elastic forces of the new positions with
//    neighbour values exchanged between adjacent lanes (DPP lane shifts), so
//    forces need no extra barrier.  Halo lanes repeat their neighbour
//    window's arithmetic bit for bit and only the 60 inner lanes publish.
// ---------------------------------------------------------------------------

// value of lane l+1 (wave_shl:1); the last lane reads 0
__device__ __forceinline__ float lane_next(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xF, 0xF, false));
}
// value of lane l-1 (wave_shr:1); lane 0 reads 0
__device__ __forceinline__ float lane_prev(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ double lane_next(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x130, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x130, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane_prev(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x138, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x138, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}


template <typename T> struct FwdLds {
    TabSys* tab;   // FP32 kernel table (FP32 runs; its index window where fwd_window)
    Src4<T>* src;  // [2 NMAX] positions (hi part) and forces, each block of 64 twice
    V2<T>* part;   // [WPS][NMAX] partial velocities
    int* bad;      // [WPS] wave flags: 1 non-finite position, 2 beyond the bound
    V2<double>* trig;  // FP64: (cos, sin) of omega t per filament, this step's and the next one's
};

constexpr int FWD_WIN = 60;  // points published per point-phase window
// Most windows one lane carries.  A single wave with all nine windows of a
// 512-point system needs over 400 registers; that build gave FP32 results
// off by up to 1e-3 (and one run past the position bound) while every
// launch shape with at most five windows per lane matches FP64, so such
// launches take more waves instead.
constexpr int FWD_MAX_WINDOWS = 5;

// per-lane state of one window of the point phase
enum : int { FL_HELD = 1, FL_OWN = 2, FL_SEG = 4, FL_NODE = 8, FL_HEAD = 16 };

// Elastic force on the point of this lane (Appendix EFT, EFB, curva: the same
// discrete energy and the same operation order as point_force): the lane
// computes the tension of its segment (to the next point) and the curvature
// terms of its own node, and takes its neighbours' through lane shifts.  The
// stretching and bending terms of one point cancel to a small remainder, so
// they are accumulated with fused multiply-adds of unrounded products, node
// p-1, p, p+1 in turn.  k0 = preferred curvature of this lane's node now.
template <typename T>
__device__ __forceinline__ void lane_force(int fl, T xh, T yh, T xl, T yl, T ss2, T sb2, T k0, T ds, T ds2, T inv2ds,
                                           T invds2, T& Fx, T& Fy)
{
    constexpr bool COMP = sizeof(T) == 4;
    const bool segv = fl & FL_SEG, nodev = fl & FL_NODE;
    T dx = lane_next(xh) - xh, dy = lane_next(yh) - yh;
    if constexpr (COMP) {
        dx += lane_next(xl) - xl;
        dy += lane_next(yl) - yl;
    }
    dx = segv ? dx : (T)0;
    dy = segv ? dy : (T)0;
    // stretching: F_i = tau_i - tau_{i-1}, tau_k = ct_k d_k with
    // ct = 2 S_s (l/ds - 1) / l.  FP32 forms the strain as
    // (l^2 - ds^2) / ((l + ds) ds), free of the cancellation in l/ds - 1, with
    // hardware reciprocals (the divisions are not ill-conditioned); FP64
    // follows point_force exactly.
    T ct;
    if constexpr (COMP) {
        const float t2 = segv ? fmaf(dx, dx, dy * dy) : 1.0f;
        const float rl = __builtin_amdgcn_rsqf(t2);
        const float l = t2 * rl;
        const float num = fmaf(dx, dx, fmaf(dy, dy, -ds2));
        ct = ss2 * num * __builtin_amdgcn_rcpf((l + ds) * ds) * rl;
    } else {
        const T l = segv ? sqrt_t(fma_t(dx, dx, dy * dy)) : (T)1;
        ct = ss2 * (l / ds - (T)1) / l;
    }
    const T txm = lane_prev(ct * dx), tym = lane_prev(ct * dy);
    const T dxm = lane_prev(dx), dym = lane_prev(dy);
    // bending: curvature node i from segments i-1 and i
    const T a = (dx + dxm) * inv2ds;
    const T bb = (dy + dym) * inv2ds;
    const T pp = (dx - dxm) * invds2;
    const T qq = (dy - dym) * invds2;
    const T S = nodev ? fma_t(a, a, bb * bb) : (T)1;
    T rS, rS32;  // 1/S, S^(-3/2)
    if constexpr (COMP) {
        const float rs = __builtin_amdgcn_rsqf(S);
        rS = rs * rs;
        rS32 = rS * rs;
    } else {
        rS = (T)1 / S;
        rS32 = rS / sqrt_t(S);
    }
    const T num = fma_t(qq, a, -pp * bb);
    const T kap = num * rS32;
    const T co = nodev ? sb2 * (kap - k0) * ds : (T)0;
    const T n3 = (T)3 * num * rS32 * rS;
    const T dka = qq * rS32 - a * n3;
    const T dkb = -pp * rS32 - bb * n3;
    const T dkp = -bb * rS32;
    const T dkq = a * rS32;
    // dkappa_i/dX for the points i-1 (A), i (B), i+1 (C)
    const T gAx = nodev ? fma_t(-dka, inv2ds, dkp * invds2) : (T)0;
    const T gAy = nodev ? fma_t(-dkb, inv2ds, dkq * invds2) : (T)0;
    const T gBx = nodev ? (T)-2 * dkp * invds2 : (T)0;
    const T gBy = nodev ? (T)-2 * dkq * invds2 : (T)0;
    const T gCx = nodev ? fma_t(dka, inv2ds, dkp * invds2) : (T)0;
    const T gCy = nodev ? fma_t(dkb, inv2ds, dkq * invds2) : (T)0;
    const T cop = lane_prev(co), gCxp = lane_prev(gCx), gCyp = lane_prev(gCy);  // node i-1
    const T con = lane_next(co), gAxn = lane_next(gAx), gAyn = lane_next(gAy);  // node i+1
    Fx = fma_t(ct, dx, -txm);
    Fy = fma_t(ct, dy, -tym);
    Fx = fma_t(-cop, gCxp, Fx);
    Fy = fma_t(-cop, gCyp, Fy);
    Fx = fma_t(-co, gBx, Fx);
    Fy = fma_t(-co, gBy, Fy);
    Fx = fma_t(-con, gAxn, Fx);
    Fy = fma_t(-con, gAyn, Fy);
}

template <typename T, int TPL, int WPS, bool AHEAD>
__device__ void run_system(const Batch& b, const Run& r, int s, const FwdLds<T>& L, T* obs, T* speed,
                           int32_t* status, int32_t* steps_done, bool refuse)
{
    constexpr bool COMP = sizeof(T) == 4;
    constexpr int NMAX = 64 * TPL, NT = 64 * WPS;
    constexpr int NWIN = (NMAX + FWD_WIN - 1) / FWD_WIN, OWNW = (NWIN + WPS - 1) / WPS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: scalar loops and branches
    const int N = b.npt[s];
    const int nsw = b.nswim[s];
    const int n = N * nsw;
    const int64_t f0 = b.sw_off[s];
    if (refuse || status[s] == SWIM_ST_BADPARAM_) {
        // parameters outside the kernel's domain (or a launch that cannot
        // run, refuse): no run, NaN outputs
        for (int m = tid; m < nsw; m += NT) {
            T* q = obs + (f0 + m) * (int64_t)r.n_obs * 2;
            for (int o = 0; o < 2 * r.n_obs; ++o) q[o] = (T)NAN;
            speed[f0 + m] = (T)NAN;
        }
        if (tid == 0) {
            if (steps_done) steps_done[s] = 0;
            if (refuse) status[s] = SWIM_ST_BADPARAM_;
        }
        __syncthreads();
        return;
    }
    const SysConst<T>& C = ((const SysConst<T>*)b.sysc)[s];
    const double dsd = 1.0 / (double)(N - 1);
    constexpr bool WIN = fwd_window(COMP ? 0 : 1, TPL, WPS);
    if constexpr (WIN)
        tab_load_window((const TabSys*)b.tab + s, reinterpret_cast<unsigned char*>(L.tab), tid, NT);
    else if constexpr (COMP)
        tab_load((const TabSys*)b.tab + s, L.tab, tid, NT);
    constexpr bool LDS64 = !COMP && AHEAD;
    if constexpr (LDS64) {
        const float4* from = reinterpret_cast<const float4*>((const TabSys64*)b.tab + s);
#pragma unroll 4
        for (int i = tid; i < (int)(sizeof(TabSys64) / 16); i += NT) reinterpret_cast<float4*>(L.tab)[i] = from[i];
    }
    const int nwin = (n + FWD_WIN - 1) / FWD_WIN;
    const int pw = min(WPS, nwin);     // waves with point work
    const bool pwave = wave < pw;      // uniform within a wave
    const T ds = (T)dsd, ds2 = (T)(dsd * dsd), inv2ds = (T)(0.5 / dsd), invds2 = (T)(1.0 / (dsd * dsd));
    const T dt = (T)r.dt;
    // the pair phase of FP32 runs works on positions scaled by the table's
    // rho (an exact power of two); registers keep the unscaled state
    const T rho = COMP ? C.tr : (T)1;

    // window state: point i = 60 g + lane - 2 of window g = wave + WPS q
    T xh[OWNW], yh[OWNW], xl[OWNW], yl[OWNW], ss2[OWNW], sb2[OWNW], ka[OWNW], kb[OWNW];
    double rc[OWNW], rs[OWNW], cd[OWNW], sd[OWNW];  // cos, sin of omega t; rotation by omega dt
    int fl[OWNW], fil[OWNW];
#pragma unroll
    for (int q = 0; q < OWNW; ++q) {
        const int g = wave + WPS * q;
        const int i = FWD_WIN * g + lane - 2;
        const bool held = g < nwin && i >= 0 && i < n;
        const int m = held ? i / N : 0, p = held ? i - m * N : 0;
        fil[q] = m;
        const double* P = b.params + 9 * (f0 + m);
        const double X = held ? P[7] + (double)p * dsd : 0.0, Y = held ? P[8] : 0.0;
        xh[q] = (T)X;
        yh[q] = (T)Y;
        xl[q] = COMP ? (T)(X - (double)xh[q]) : (T)0;
        yl[q] = COMP ? (T)(Y - (double)yh[q]) : (T)0;
        const bool own = held && lane >= 2 && lane < 2 + FWD_WIN;
        fl[q] = (held ? FL_HELD : 0) | (own ? FL_OWN : 0) | (held && p <= N - 2 ? FL_SEG : 0) |
                (held && p >= 1 && p <= N - 2 ? FL_NODE : 0) | (own && p == N - 1 ? FL_HEAD : 0);
        ss2[q] = (T)(2.0 * P[2]);
        sb2[q] = (T)(2.0 * P[1]);
        // kappa0_p(t) = -k^2 b sin(k s_p + phase - omega t)
        //            = ka cos(omega t) - kb sin(omega t)
        const double amp = -P[5] * P[5] * P[3], ph = P[5] * ((double)p * dsd) + P[6];
        ka[q] = (T)(amp * sin(ph));
        kb[q] = (T)(amp * cos(ph));
        rc[q] = 1.0;
        rs[q] = 0.0;
        cd[q] = COMP ? cos(P[4] * r.dt) : P[4];  // FP64 keeps omega and evaluates directly
        sd[q] = COMP ? sin(P[4] * r.dt) : 0.0;
        if (fl[q] & FL_HEAD) {
            // samples a stopped run never reaches stay NaN
            T* o = obs + (f0 + m) * (int64_t)r.n_obs * 2;
            for (int k = 0; k < 2 * r.n_obs; ++k) o[k] = (T)NAN;
        }
    }
    // early rejection (one swimmer per system): the head lane's running sum
    // of squared deviations from the data
    const bool early = r.stop_data != nullptr && nsw == 1;
    double ssq = 0.0;
    bool rejected = false;
    // FP64: a wave without point work evaluates cos and sin of omega t for the
    // next step while the point waves work on this one (in these they are 0.4 us
    // of a chain of 3.8); two buffers, by the step's parity
    const bool helped = !COMP && pw < WPS;
    auto help = [&](int next) {
        for (int m = lane; m < nsw; m += 64) {
            const double wt = b.params[9 * (f0 + m) + 4] * ((double)next * r.dt);
            V2<double> v;
            v.x = cos(wt);
            v.y = sin(wt);
            L.trig[(next & 1) * nsw + m] = v;
        }
    };
    // forces of the held points at the current time; owners publish them
    auto point_forces = [&]() {
#pragma unroll
        for (int q = 0; q < OWNW; ++q) {
            T Fx, Fy;
            const T k0 = fma_t(ka[q], (T)rc[q], -kb[q] * (T)rs[q]);
            lane_force<T>(fl[q], xh[q], yh[q], xl[q], yl[q], ss2[q], sb2[q], k0, ds, ds2, inv2ds, invds2, Fx, Fy);
            if (fl[q] & FL_OWN) {
                const int i = FWD_WIN * (wave + WPS * q) + lane - 2;
                Src4<T> v;
                v.x = xh[q] * rho;
                v.y = yh[q] * rho;
                v.fx = Fx;
                v.fy = Fy;
                const int slot = src2_slot(i);
                L.src[slot] = v;
                L.src[slot + 64] = v;
            }
        }
    };
    // points n .. 64 B - 1 of the last block: no force, at the start position of
    // point n - 1 (they add nothing and stay within the system's extent)
    for (int i = n + tid; i < 64 * ((n + 63) >> 6); i += NT) {
        const double* P = b.params + 9 * (f0 + nsw - 1);
        Src4<T> v;
        v.x = (T)(P[7] + (double)(N - 1) * dsd) * rho;
        v.y = (T)P[8] * rho;
        v.fx = (T)0;
        v.fy = (T)0;
        const int slot = src2_slot(i);
        L.src[slot] = v;
        L.src[slot + 64] = v;
    }
    if (pwave)
        point_forces();
    else if (helped && wave == WPS - 1)
        help(1);
    __syncthreads();
    int st = 0, done = r.steps;
    const int nblk64 = (n + 63) >> 6;
    // this wave's share of the pair schedule when it is one segment
    int seg_a = 0, seg_b = 0, seg_lo = 0, seg_hi = 0;
    bool one_seg = sym_one_segment<WPS>(n, wave, seg_a, seg_b, seg_lo, seg_hi);
    one_seg = __builtin_amdgcn_readfirstlane(one_seg ? 1 : 0) != 0;
    seg_a = __builtin_amdgcn_readfirstlane(seg_a);
    seg_b = __builtin_amdgcn_readfirstlane(seg_b);
    seg_lo = __builtin_amdgcn_readfirstlane(seg_lo);
    seg_hi = __builtin_amdgcn_readfirstlane(seg_hi);
    int obs_left = r.obs_every, obs_k = 0;  // steps to the next sample, its index
    for (int step = 0; step < r.steps; ++step) {
        // pair phase: this wave's share of the symmetric pair schedule
        {
            // no pair lies beyond the FP32 table: every step starts from
            // positions within the run bound |x|, |y| <= 1e3 (a step that
            // leaves it ends the run), so r <= 2829, and the host sends the
            // systems whose 2829 / eps reaches 2^22 (eps_over_ds well below
            // its usual 1.5) to the large-system step, so that here
            // 1 + (r/eps)^2 < 2^44, inside the table (the initial positions
            // are the caller's: a run placed beyond the bound reads zeros
            // for its far pairs in its first step and stops)
            // (FP64 reads its table from LDS or HBM and tests every pair)
            T ax[TPL], ay[TPL];
            const void* tab = COMP ? (const void*)L.tab : (const void*)((const TabSys64*)b.tab + s);
            constexpr int W = WIN ? (AHEAD ? 2 : 1) : LDS64 ? 4 : 0;
            if (one_seg)
                pair_phase_seg<T, TPL, !COMP, W>(C, tab, L.src, seg_a, seg_b, seg_lo, seg_hi, lane, ax, ay);
            else
                pair_phase_sym<T, TPL, WPS, !COMP, W>(C, tab, L.src, n, wave, lane, ax, ay);
#pragma unroll
            for (int c = 0; c < TPL; ++c) {
                if (c < nblk64) {
                    V2<T> v;
                    v.x = ax[c];
                    v.y = ay[c];
                    L.part[wave * NMAX + 64 * c + lane] = v;
                }
            }
        }
        __syncthreads();
        // point phase: Euler step of the held points, forces at t_{step+1}
        if (pwave) {
            int bad = 0;
#pragma unroll
            for (int q = 0; q < OWNW; ++q) {
                if (fl[q] & FL_HELD) {
                    const int i = FWD_WIN * (wave + WPS * q) + lane - 2;
                    // all partials in flight at once, then summed in wave order
                    V2<T> pv[WPS];
#pragma unroll
                    for (int w = 0; w < WPS; ++w) pv[w] = L.part[w * NMAX + i];
                    T ux = (T)0, uy = (T)0;
#pragma unroll
                    for (int w = 0; w < WPS; ++w) {
                        ux += pv[w].x;
                        uy += pv[w].y;
                    }
                    if constexpr (COMP) {
                        acc2(xh[q], xl[q], dt * ux);
                        acc2(yh[q], yl[q], dt * uy);
                    } else {
                        xh[q] = fma_t(dt, ux, xh[q]);
                        yh[q] = fma_t(dt, uy, yh[q]);
                    }
                    if ((fl[q] & FL_OWN) && (bad_t(xh[q]) || bad_t(yh[q])))
                        bad |= isfinite(xh[q]) && isfinite(yh[q]) ? 2 : 1;
                }
                if constexpr (COMP) {
                    const double c = rc[q], sn = rs[q];
                    rc[q] = fma(c, cd[q], -sn * sd[q]);
                    rs[q] = fma(sn, cd[q], c * sd[q]);
                } else if (helped) {
                    const V2<double> v = L.trig[((step + 1) & 1) * nsw + fil[q]];
                    rc[q] = v.x;
                    rs[q] = v.y;
                } else {
                    const double wt = cd[q] * ((double)(step + 1) * r.dt);
                    rc[q] = cos(wt);
                    rs[q] = sin(wt);
                }
            }
            point_forces();
            bad |= rejected ? 4 : 0;
            int flags = 0;
            if (__any(bad))
                flags = (__any(bad & 1) ? 1 : 0) | (__any(bad & 2) ? 2 : 0) | (__any(bad & 4) ? 4 : 0);
            if (lane == 0) L.bad[wave] = flags;
        } else if (helped && wave == WPS - 1) {
            help(step + 2);
        }
        __syncthreads();
        // the point waves' flags, one per lane, combined by ballot (uniform)
        const int bw = lane < pw ? L.bad[lane] : 0;
        if (__any(bw)) {
            st = __any(bw & 1) ? 1 : __any(bw & 2) ? 2 : SWIM_ST_REJECTED_;
            done = step + 1;
            break;
        }
        if (r.obs_every > 0 && --obs_left == 0) {
            obs_left = r.obs_every;
            const int o = obs_k++;
            if (pwave) {
#pragma unroll
                for (int q = 0; q < OWNW; ++q) {
                    if (fl[q] & FL_HEAD) {
                        const int i = FWD_WIN * (wave + WPS * q) + lane - 2;
                        T* d = obs + ((f0 + i / N) * (int64_t)r.n_obs + o) * 2;
                        const T hx = xh[q] + xl[q], hy = yh[q] + yl[q];
                        d[0] = hx;
                        d[1] = hy;
                        if (early) {
                            const double ex = (double)hx - r.stop_data[2 * o];
                            const double ey = (double)hy - r.stop_data[2 * o + 1];
                            ssq = fma(ex, ex, fma(ey, ey, ssq));
                            rejected = ssq > r.stop_ssq;
                        }
                    }
                }
            }
        }
    }
    if (pwave) {
        const T Tend = (T)((double)r.steps * r.dt);
#pragma unroll
        for (int q = 0; q < OWNW; ++q) {
            if (fl[q] & FL_HEAD) {
                const int i = FWD_WIN * (wave + WPS * q) + lane - 2;
                const int64_t f = f0 + i / N;
                if (st) {
                    speed[f] = (T)NAN;
                } else {
                    const T hx0 = (T)(b.params[9 * f + 7] + (double)(N - 1) * dsd);
                    const T hy0 = (T)b.params[9 * f + 8];
                    const T dx = (xh[q] + xl[q]) - hx0, dy = (yh[q] + yl[q]) - hy0;
                    speed[f] = sqrt_t(fma_t(dx, dx, dy * dy)) / Tend;
                }
            }
        }
    }
    if (tid == 0) {
        status[s] = st;
        if (steps_done) steps_done[s] = done;
    }
    __syncthreads();
}

// FP32 systems of up to 128 points in 16-wave workgroups are held to 64
// VGPRs (8 waves per SIMD): two systems then share a CU, so that one's
// barriers and LDS latency overlap the other's pair phase (without the
// bound the build takes 92 VGPRs and one system per CU; the spills the bound
// costs lie outside the pair loop).  AHEAD: FP32, the pair loop on the table
// window reads ahead, up to 128 points where no workgroup shares a CU (a build of
// its own: 48 runs of 128 points 1251 us against 1287, but 4096 of them 11.07 ms
// against 10.45; above 128 points, 16 waves, it gives nothing: 600 runs of 512
// points, 200 steps, 15.4 against 15.1 ms); FP64, the table in LDS (fwd_lds64).
template <typename T, int TPL, int WPS, bool AHEAD = false>
__global__ __launch_bounds__(64 * WPS) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && TPL <= 2 && WPS == 16
                                                                                 ? 8
                                                                                 : 1))) void
k_forward(Batch b, Run r, const int32_t* order, int32_t* queue, T* obs, T* speed, int32_t* status, int32_t* steps_done)
{
    extern __shared__ __align__(16) unsigned char smem[];
    FwdLds<T> L;
    const FwdLdsLayout lay = fwd_lds_layout(sizeof(T) == 4 ? 0 : 1, TPL, WPS, sizeof(T) == 8 && AHEAD);
    L.tab = reinterpret_cast<TabSys*>(smem + lay.tab);
    L.src = reinterpret_cast<Src4<T>*>(smem + lay.src);
    L.part = reinterpret_cast<V2<T>*>(smem + lay.part);
    L.bad = reinterpret_cast<int*>(smem + lay.bad);
    L.trig = reinterpret_cast<V2<double>*>(smem + lay.trig);
    int& s_item = L.bad[WPS];
    // the pair loop of the index-window layout addresses the table from LDS
    // address 0, where the dynamic LDS starts while the kernel declares no
    // static LDS; should it start elsewhere, every system is refused
    // (status SWIM_ST_BADPARAM, NaN outputs) rather than run on wrong data
    bool refuse = false;
#if defined(__HIP_DEVICE_COMPILE__)
    refuse = (fwd_window(sizeof(T) == 4 ? 0 : 1, TPL, WPS) || (sizeof(T) == 8 && AHEAD)) &&
             (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)smem != 0u;
#endif
    // Instruction-issue priority of this launch's waves against the other
    // size buckets' launches that share its CUs: larger systems first.  A
    // system's run costs ~N^2 per step, so in an uneven batch the largest
    // runs that do not stop early set the call's length; a SIMD picks the
    // highest-priority ready wave, and the smaller systems' waves take the
    // slots those leave idle (barriers, LDS latency).
    __builtin_amdgcn_s_setprio(TPL >= 6 ? 3 : TPL >= 4 ? 2 : TPL >= 2 ? 1 : 0);
    // Work queue: thread 0 takes the next system; the item reaches every
    // thread through LDS and readfirstlane makes it an SGPR, so the loop exit
    // is a uniform scalar branch.  A workgroup takes at most n_sys items.
    for (int64_t it = 0; it <= b.n_sys; ++it) {
        if (threadIdx.x == 0) s_item = atomicAdd(queue, 1);
        __syncthreads();
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        if (item >= b.n_sys) break;
        const int s = __builtin_amdgcn_readfirstlane(order[item]);
        run_system<T, TPL, WPS, AHEAD>(b, r, s, L, obs, speed, status, steps_done, refuse);
    }
}

// ---------------------------------------------------------------------------
// large systems: one launch per step, targets split over workgroups; every
// workgroup rebuilds the forces of the whole system, tile by tile, into LDS
// (O(N) work next to its O(N * 256 * TPL) pair work), positions are
// double-buffered in HBM.  The LDS holds the table and one tile of sources,
// so any system size fits and two workgroups share a CU.
// ---------------------------------------------------------------------------
constexpr int BIG_TILE = 1024;  // sources per LDS tile
template <typename T>
__global__ void k_big_init(const int64_t* list, Batch b, BigState S, int32_t* status, T* obs, int32_t n_obs)
{
    constexpr bool COMP = sizeof(T) == 4;
    const int64_t s = list[blockIdx.y];
    const int64_t p0 = b.pt_off[s];
    const int N = b.npt[s];
    const int n = N * b.nswim[s];
    if (status[s] == SWIM_ST_BADPARAM_) {
        for (int m = blockIdx.x * blockDim.x + threadIdx.x; m < b.nswim[s]; m += gridDim.x * blockDim.x) {
            const int64_t f = b.sw_off[s] + m;
            for (int o = 0; o < 2 * n_obs; ++o) obs[f * (int64_t)n_obs * 2 + o] = (T)NAN;
        }
        return;
    }
    const double dsd = 1.0 / (double)(N - 1);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int m = i / N, p = i - m * N;
        const int64_t f = b.sw_off[s] + m;
        const double X = b.params[9 * f + 7] + (double)p * dsd;
        const double Y = b.params[9 * f + 8];
        const T xh = (T)X, yh = (T)Y;
        ((T*)S.xh[0])[p0 + i] = xh;
        ((T*)S.yh[0])[p0 + i] = yh;
        ((T*)S.xl[0])[p0 + i] = COMP ? (T)(X - (double)xh) : (T)0;
        ((T*)S.yl[0])[p0 + i] = COMP ? (T)(Y - (double)yh) : (T)0;
        if (p == N - 1) {
            ((T*)S.head0)[2 * f] = (T)X;
            ((T*)S.head0)[2 * f + 1] = (T)Y;
            for (int o = 0; o < 2 * n_obs; ++o) obs[f * (int64_t)n_obs * 2 + o] = (T)NAN;
        }
    }
}

// source record of point i of a large system at time t: its position (hi
// part) and elastic force, from the positions of the current buffer
template <typename T>
__device__ __forceinline__ Src4<T> big_source(const Batch& b, const T* xh, const T* yh, const T* xl, const T* yl,
                                              int64_t f0, int N, int i, T t)
{
    constexpr bool COMP = sizeof(T) == 4;
    const int m = i / N, p = i - m * N;
    const FilP<T> q = load_filp<T>(b.params, f0 + m, N);
    const int base = m * N;
    auto seg = [&](int kk, T& dx, T& dy) {
        const int a = base + kk, c = base + kk + 1;
        dx = (xh[c] - xh[a]) + (COMP ? xl[c] - xl[a] : (T)0);
        dy = (yh[c] - yh[a]) + (COMP ? yl[c] - yl[a] : (T)0);
    };
    T Fx, Fy;
    point_force<T>(seg, p, q, t, Fx, Fy);
    Src4<T> v;
    v.x = xh[i];
    v.y = yh[i];
    v.fx = Fx;
    v.fy = Fy;
    return v;
}

// Euler step of point i of a large system from its velocity (ux, uy):
// position (hi, lo) into buffer nxt, the bound check, the head sample
template <typename T>
__device__ __forceinline__ void big_update_point(const BigState& S, int step, const Run& r, int64_t s, int64_t p0,
                                                 int64_t f0, int N, int64_t i, int nxt, T hx, T hy, T lx, T ly, T ux,
                                                 T uy, T* obs, int32_t* status, int32_t* steps_done)
{
    constexpr bool COMP = sizeof(T) == 4;
    const T dt = (T)r.dt;
    if (COMP) {
        acc2(hx, lx, dt * ux);
        acc2(hy, ly, dt * uy);
    } else {
        hx = fma_t(dt, ux, hx);
        hy = fma_t(dt, uy, hy);
    }
    ((T*)S.xh[nxt])[p0 + i] = hx;
    ((T*)S.yh[nxt])[p0 + i] = hy;
    ((T*)S.xl[nxt])[p0 + i] = lx;
    ((T*)S.yl[nxt])[p0 + i] = ly;
    if (bad_t(hx) || bad_t(hy)) {
        atomicMax(&status[s], (isfinite(hx) && isfinite(hy)) ? 2 : 1);
        if (steps_done) steps_done[s] = step + 1;
    }
    if (r.obs_every > 0 && (step + 1) % r.obs_every == 0) {
        const int m = (int)(i / N), p = (int)(i - (int64_t)m * N);
        if (p == N - 1) {
            const int o = (step + 1) / r.obs_every - 1;
            T* q = obs + ((f0 + m) * (int64_t)r.n_obs + o) * 2;
            q[0] = hx + lx;
            q[1] = hy + ly;
        }
    }
}

template <typename T, int TPL>
__global__ __launch_bounds__(256) void k_big_step(const int64_t* blk_sys, const int64_t* blk_first, Batch b,
                                                  BigState S, int step, Run r, T* obs, int32_t* status,
                                                  int32_t* steps_done)
{
    constexpr bool COMP = sizeof(T) == 4;
    constexpr size_t TABB = COMP ? sizeof(TabSys) : 0;
    extern __shared__ __align__(16) unsigned char smem[];
    TabSys* tab = reinterpret_cast<TabSys*>(smem);
    Src4<T>* src = reinterpret_cast<Src4<T>*>(smem + TABB);  // [BIG_TILE]
    __shared__ int s_status;
    const int tid = threadIdx.x;
    const int64_t s = blk_sys[blockIdx.x];
    // one read of the status per workgroup (other workgroups of this launch
    // may raise it meanwhile), broadcast through LDS so that every wave
    // takes the same exit before the barriers below
    if (tid == 0) s_status = status[s];
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_status) != 0) return;
    if constexpr (COMP) tab_load((const TabSys*)b.tab + s, tab, tid, 256);
    const int64_t first = blk_first[blockIdx.x];
    const int64_t p0 = b.pt_off[s];
    const int N = b.npt[s];
    const int n = N * b.nswim[s];
    const int64_t f0 = b.sw_off[s];
    const int cur = step & 1, nxt = cur ^ 1;
    const T* xh = (const T*)S.xh[cur] + p0;
    const T* yh = (const T*)S.yh[cur] + p0;
    const T* xl = (const T*)S.xl[cur] + p0;
    const T* yl = (const T*)S.yl[cur] + p0;
    const T t = (T)((double)step * r.dt);
    const SysConst<T>& C = ((const SysConst<T>*)b.sysc)[s];
    // FP32 sums whole large systems per lane: FP64 accumulation
    // (pair_accumulate_x); FP64 runs accumulate in FP64 anyway
    T xi[TPL], yi[TPL], ax[TPL], ay[TPL];
    double axd[TPL], ayd[TPL];
#pragma unroll
    for (int k = 0; k < TPL; ++k) {
        const int64_t i = first + tid + 256 * k;
        xi[k] = i < n ? xh[i] : (T)0;
        yi[k] = i < n ? yh[i] : (T)0;
        ax[k] = ay[k] = (T)0;
        axd[k] = ayd[k] = 0.0;
    }
    // sources in tiles of BIG_TILE: the forces of a tile's points (read
    // positions only) into LDS, then every target of this workgroup sums
    // over them
    for (int j0 = 0; j0 < n; j0 += BIG_TILE) {
        const int m_t = min(BIG_TILE, n - j0);
        if (j0 > 0) __syncthreads();  // the previous tile is consumed
        for (int jj = tid; jj < m_t; jj += 256) src[jj] = big_source<T>(b, xh, yh, xl, yl, f0, N, j0 + jj, t);
        __syncthreads();
        if constexpr (COMP)
            pair_accumulate_x<TPL>(C, tab, src, m_t, xi, yi, axd, ayd);
        else
            pair_accumulate<T, TPL>(C, (const TabSys64*)b.tab + s, src, m_t, xi, yi, ax, ay);
    }
#pragma unroll
    for (int k = 0; k < TPL; ++k) {
        const int64_t i = first + tid + 256 * k;
        if (i >= n) continue;
        const T ux = COMP ? (T)axd[k] : ax[k];
        const T uy = COMP ? (T)ayd[k] : ay[k];
        big_update_point<T>(S, step, r, s, p0, f0, N, i, nxt, xi[k], yi[k], xl[i], yl[i], ux, uy, obs, status,
                            steps_done);
    }
}

// ---------------------------------------------------------------------------
// large systems in FP32, symmetric: every pair of points is evaluated once
// and serves both ends, in forward steps and in velocity sums of given
// forces.  Points form tiles of 128 (two blocks of 64); one workgroup of
// four waves takes one pair of tiles (ta <= tb) of one system.  A wave holds
// a block of tile ta as targets, one point per lane, and runs over a block of
// tile tb (its own or a later one when ta == tb) with the lane schedule of
// the small systems: at offset s lane l pairs its target with point (l + s) mod 64 of
// the block, whose sums rotate down one lane per offset.  Both ends accumulate in FP64 as in
// pair_accumulate_x (the constant part of Ht in two floats, exact products).
// The workgroup leaves tile ta's sums over tile tb and tile tb's over tile
// ta in two slots of a partial-sum buffer (one slot when ta == tb); then
// k_big_update adds a tile's slots in a fixed order and takes the Euler
// step: deterministic, no atomics on the sums.
// ---------------------------------------------------------------------------

// offsets [s_lo, s_hi) of one block pair: ti is this lane's target (its
// force in FP64: tfx, tfy), sp + lane + s the moving point at offset s (the
// block stored twice).  Targets' sums add to (ax, ay); the moving points'
// sums of this pass return in (bxo, byo), realigned to lane = point.  Offsets
// from s_full on (the diagonal block's offset 32) count for lanes 0..31
// only.  FAR: only the pairs beyond the table, evaluated directly.
template <bool FAR>
__device__ __forceinline__ bool big_sym_block(const SysConst<float>& C, const TabSys* tab, const Src4<float>& ti,
                                              double tfx, double tfy, const Src4<float>* sp, int s_lo, int s_full,
                                              int s_hi, int lane, double& ax, double& ay, double& bxo, double& byo)
{
    const float ts = C.ts;
    double bx = 0.0, by = 0.0;
    bool far = false;
    auto offset = [&](const Src4<float>& q, bool live) {
        const float dx = ti.x - q.x, dy = ti.y - q.y;
        const float t = fmaf(dx, dx, dy * dy);
        const uint32_t bits = tab_bits(t, ts);
        const uint32_t id = bits >> TAB_SHIFT;
        float h0, lo, H2;
        if constexpr (!FAR) {
            far = far || id >= TAB_END;
            const uint32_t ic = min(id, TAB_END) - TAB_BIAS;
            const TabE& e = tab->e[ic];
            const float u = tab_u(bits);
            h0 = e.h[0];
            lo = tab->h0lo[ic] + u * fmaf(fmaf(e.h[3], u, e.h[2]), u, e.h[1]);
            H2 = fmaf(fmaf(fmaf(e.g[3], u, e.g[2]), u, e.g[1]), u, e.g[0]) * ts;
        } else {
            h0 = 0.0f;
            lo = 0.0f;
            H2 = 0.0f;
            if (id >= TAB_END) kernel_eval<float>(C, t, h0, H2);
        }
        if (!live) {
            h0 = 0.0f;
            lo = 0.0f;
            H2 = 0.0f;
        }
        // h0 + lo is exact in FP64
        const double hd = (double)h0 + (double)lo;
        const double dxd = dx, dyd = dy, qfx = q.fx, qfy = q.fy;
        const double fdj = (double)(H2 * fmaf(q.fx, dx, q.fy * dy));
        const double fdi = (double)(H2 * fmaf(ti.fx, dx, ti.fy * dy));
        ax = fma(hd, qfx, fma(fdj, dxd, ax));
        ay = fma(hd, qfy, fma(fdj, dyd, ay));
        bx = lane_rot(fma(hd, tfx, fma(fdi, dxd, bx)));
        by = lane_rot(fma(hd, tfy, fma(fdi, dyd, by)));
    };
    const Src4<float>* spl = sp + lane;
    int s = __builtin_amdgcn_readfirstlane(s_lo);
    const int sf = __builtin_amdgcn_readfirstlane(s_full);
    for (; s + 1 < sf; s += 2) {
        offset(spl[s], true);
        offset(spl[s + 1], true);
    }
    if (s < sf) offset(spl[s], true);
    if (sf < s_hi) offset(spl[sf], lane < 32);
    // lane l now holds the sums of point (l + s_hi) mod 64 of the block
    const int from = (lane - s_hi) & 63;
    bxo = __shfl(bx, from, 64);
    byo = __shfl(by, from, 64);
    return far;
}

constexpr int BT = BIG_TILE_POINTS;  // points per tile: two blocks
static_assert(BT == 128, "four waves, one per block pair of two tiles");

// LDS of k_tile_pairs: [table][tile ta][tile tb, each block twice][sums of
// tile tb's points by block of ta][sums of tile ta's points by block of tb]
struct TileLds {
    static constexpr size_t src = sizeof(TabSys), src2 = src + BT * sizeof(Src4<float>),
                            pb = src2 + 2 * BT * sizeof(Src4<float>), pa = pb + 2 * BT * sizeof(V2<double>),
                            total = pa + 2 * BT * sizeof(V2<double>);
};
static_assert(sizeof(TabSys) % 16 == 0, "16-byte aligned LDS sections");

// One workgroup of four waves per tile pair (ta <= tb) of one system, one wave
// per block pair: the off-diagonal pairs of all systems first, then the
// diagonal ones (three quarters of the work, so that they fill the launch's
// tail).  Sources: bt.src (position, force), or x, y, fx, fy (SOA).  40 KB of
// LDS: four workgroups share a CU, one's table copy and sums overlapping the
// others' pair loops.  Bound by VALU issue (47.5 operations per pair and
// both ends, FP64 accumulation among them).  Tiles of 256 points (a wave per
// block of ta running over four blocks of tb, three workgroups a CU) took 832
// us against 702 for a velocity sum of 64 x 4096 points, and 49 against 30 us
// for the step of two such systems, whose 272 pairs leave most of the chip idle.
template <bool SOA>
__global__ __launch_bounds__(256) void k_tile_pairs(BigTiles bt, const SysConst<float>* sysc, const TabSys* tabs,
                                                    const float* x, const float* y, const float* fx, const float* fy,
                                                    const int32_t* status)
{
    using L = TileLds;
    extern __shared__ __align__(16) unsigned char smem[];
    TabSys* tab = reinterpret_cast<TabSys*>(smem);
    Src4<float>* sa = reinterpret_cast<Src4<float>*>(smem + L::src);
    Src4<float>* sb2 = reinterpret_cast<Src4<float>*>(smem + L::src2);
    V2<double>* pb = reinterpret_cast<V2<double>*>(smem + L::pb);
    V2<double>* pa = reinterpret_cast<V2<double>*>(smem + L::pa);
    __shared__ int s_status;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // which system and tiles
    const int64_t n_off = bt.off0[bt.n_big];
    int64_t g;
    int ta, tb;
    if ((int64_t)blockIdx.x < n_off) {
        g = prefix_item(bt.off0, bt.n_big, blockIdx.x);
        const int64_t k = (int64_t)blockIdx.x - bt.off0[g];  // pair k: tb (tb - 1) / 2 + ta, ta < tb
        int64_t t = (int64_t)(0.5 * (1.0 + sqrt(1.0 + 8.0 * (double)k)));
        while (t * (t - 1) / 2 > k) --t;
        while (t * (t + 1) / 2 <= k) ++t;
        tb = (int)t;
        ta = (int)(k - t * (t - 1) / 2);
    } else {
        g = prefix_item(bt.tile0, bt.n_big, (int64_t)blockIdx.x - n_off);
        ta = tb = (int)((int64_t)blockIdx.x - n_off - bt.tile0[g]);
    }
    const int64_t s = bt.list[g];
    if (status) {
        // one read of the status per workgroup, broadcast (uniform exit)
        if (tid == 0) s_status = status[s];
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(s_status) != 0) return;
    }
    tab_load(tabs + s, tab, tid, 256);
    const int64_t p0 = bt.pt0[g];
    const int n = bt.cnt[g], nt = (n + BT - 1) / BT;
    const SysConst<float>& C = sysc[s];
    const bool diag = ta == tb;
    // sources of both tiles; points beyond n: at point n - 1, no force (they
    // add nothing and their own sums are not used)
    auto source = [&](int i) {
        const int64_t k = p0 + min(i, n - 1);
        Src4<float> v;
        if constexpr (SOA) {
            v.x = x[k];
            v.y = y[k];
            v.fx = fx[k];
            v.fy = fy[k];
        } else {
            v = reinterpret_cast<const Src4<float>*>(bt.src)[k];
        }
        if (i >= n) v.fx = v.fy = 0.0f;
        return v;
    };
    // the first two waves load tile tb, the others tile ta
    const int jj = tid & (BT - 1);
    if (tid < BT) {
        const Src4<float> v = source(tb * BT + jj);
        const int k = src2_slot(jj);
        sb2[k] = v;
        sb2[k + 64] = v;
    } else if (!diag) {
        sa[jj] = source(ta * BT + jj);
    }
    __syncthreads();
    const int a = w >> 1, bb = w & 1;  // this wave's block pair
    const Src4<float> ti = diag ? sb2[(a << 7) + lane] : sa[(a << 6) + lane];
    const double tfx = ti.fx, tfy = ti.fy;
    double ax = 0.0, ay = 0.0, bx = 0.0, by = 0.0;
    if (!diag || bb >= a) {
        // the diagonal block: offsets 1..32, offset 32 for lanes 0..31
        const bool dblk = diag && bb == a;
        const int s_lo = dblk ? 1 : 0, s_full = dblk ? 32 : 64, s_hi = dblk ? 33 : 64;
        const Src4<float>* sp = sb2 + (bb << 7);
        const bool far = big_sym_block<false>(C, tab, ti, tfx, tfy, sp, s_lo, s_full, s_hi, lane, ax, ay, bx, by);
        if (__any(far)) {
            double fx2, fy2;
            big_sym_block<true>(C, tab, ti, tfx, tfy, sp, s_lo, s_full, s_hi, lane, ax, ay, fx2, fy2);
            bx += fx2;
            by += fy2;
        }
    }
    pb[a * BT + (bb << 6) + lane] = V2<double>{bx, by};
    pa[bb * BT + (a << 6) + lane] = V2<double>{ax, ay};
    __syncthreads();
    // slot (t, q): tile t's sums over tile q; a diagonal pair's two kinds of
    // sums share one slot
    V2<double>* const pbuf = reinterpret_cast<V2<double>*>(bt.part) + bt.slot0[g] * BT;
    if (tid < BT) {
        V2<double> u = pb[tid], v = pa[tid];
        u.x += pb[BT + tid].x;
        u.y += pb[BT + tid].y;
        v.x += pa[BT + tid].x;
        v.y += pa[BT + tid].y;
        if (diag) {
            u.x += v.x;
            u.y += v.y;
        } else {
            pbuf[((int64_t)ta * nt + tb) * BT + tid] = v;
        }
        pbuf[((int64_t)tb * nt + ta) * BT + tid] = u;
    }
}

// the velocities of the tile-pair path for given forces: a point's slots in
// tile order, and H1(0) times the sum of the forces (FP64: they cancel)
__global__ __launch_bounds__(256) void k_tile_velocity(BigTiles bt, const SysConst<float>* sysc, const float* fx,
                                                       const float* fy, float* ux, float* uy)
{
    __shared__ double red[2][4];
    const int tid = threadIdx.x;
    const int64_t g = prefix_item(bt.tile0, bt.n_big, blockIdx.x);
    const int tile = (int)((int64_t)blockIdx.x - bt.tile0[g]);
    const int64_t p0 = bt.pt0[g];
    const int n = bt.cnt[g], nt = (n + BT - 1) / BT;
    double sfx = 0.0, sfy = 0.0;
    for (int j = tid; j < n; j += 256) {
        sfx += fx[p0 + j];
        sfy += fy[p0 + j];
    }
    sfx = wave_sum(sfx);
    sfy = wave_sum(sfy);
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = sfx;
        red[1][tid >> 6] = sfy;
    }
    __syncthreads();
    const int64_t i = (int64_t)tile * BT + tid;
    if (tid >= BT || i >= n) return;
    const V2<double>* src = reinterpret_cast<const V2<double>*>(bt.part) + (bt.slot0[g] + (int64_t)tile * nt) * BT + tid;
    double u = 0.0, v = 0.0;
    for (int q = 0; q < nt; ++q) {
        const V2<double> e = src[(int64_t)q * BT];
        u += e.x;
        v += e.y;
    }
    const double h1c = sysc[bt.list[g]].h1c;
    ux[p0 + i] = (float)fma(h1c, red[0][0] + red[0][1] + red[0][2] + red[0][3], u);
    uy[p0 + i] = (float)fma(h1c, red[1][0] + red[1][1] + red[1][2] + red[1][3], v);
}

// The tile-pair path's sums without its partial-sum buffer, bit for bit: for
// callers that cannot allocate it (swim_pair_velocity_noalloc) and systems below
// its size.  One-sided: a workgroup takes a block of 64 targets, one per lane,
// and its eight waves each a block of sources at a time, in the lane schedule and
// with the code of the block pair it is there, target block (of the lower tile)
// or moving one; the blocks' sums join by tile in k_tile_pairs' order, the tiles
// in k_tile_velocity's.  Bound by VALU issue; every pair is evaluated for each of
// its ends: 4 x 4096 points 141 us a call against 105 with the buffer.
// blk0[s]: first workgroup of system s.
struct OrderedLds {
    TabSys tab;
    Src4<float> own[128], src[VEL_WAVES][128];  // each block twice
    V2<double> part[VEL_WAVES][64], diag[64];
    double red[2][4];
};
__global__ __launch_bounds__(64 * VEL_WAVES) void k_ordered_velocity(int64_t n_sys, const int64_t* blk0,
                                                                     const int64_t* pt_off,
                                                                     const SysConst<float>* sysc, const TabSys* tabs,
                                                                     const float* x, const float* y, const float* fx,
                                                                     const float* fy, float* ux, float* uy)
{
    __shared__ __align__(16) unsigned char smem[sizeof(OrderedLds)];
    OrderedLds& L = *reinterpret_cast<OrderedLds*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t s = prefix_item(blk0, n_sys, blockIdx.x);
    const int64_t p0 = pt_off[s];
    const int n = (int)(pt_off[s + 1] - p0), nt = (n + BT - 1) / BT;
    const int A = (int)((int64_t)blockIdx.x - blk0[s]), tA = A >> 1;  // this workgroup's block, its tile
    const SysConst<float>& C = sysc[s];
    tab_load(tabs + s, &L.tab, tid, 64 * VEL_WAVES);
    // point 64 k + lane; beyond n: at point n - 1, no force
    auto point = [&](int k) {
        const int i = 64 * k + lane;
        const int64_t j = p0 + min(i, n - 1);
        Src4<float> v;
        v.x = x[j];
        v.y = y[j];
        v.fx = i < n ? fx[j] : 0.0f;
        v.fy = i < n ? fy[j] : 0.0f;
        return v;
    };
    const Src4<float> own = point(A);
    if (w == 0) L.own[lane] = L.own[lane + 64] = own;
    if (w < 4) {  // the forces' sum as in k_tile_velocity
        double sfx = 0.0, sfy = 0.0;
        for (int j = tid; j < n; j += 256) {
            sfx += fx[p0 + j];
            sfy += fy[p0 + j];
        }
        sfx = wave_sum(sfx);
        sfy = wave_sum(sfy);
        if (lane == 0) {
            L.red[0][w] = sfx;
            L.red[1][w] = sfy;
        }
    }
    double u = 0.0, v = 0.0;
    for (int k0 = 0; k0 < 2 * nt; k0 += VEL_WAVES) {
        const int k = k0 + w;
        Src4<float> q{};
        if (k < 2 * nt) {
            q = point(k);
            L.src[w][lane] = L.src[w][lane + 64] = q;
        }
        __syncthreads();
        V2<double> P{0.0, 0.0};
        if (k < 2 * nt) {
            // as the target block, or as the moving one
            auto target = [&](int s_lo, int s_full, int s_hi, V2<double>& a, V2<double>* m) {
                double bx, by, cx, cy;
                const bool far = big_sym_block<false>(C, &L.tab, own, own.fx, own.fy, L.src[w], s_lo, s_full, s_hi,
                                                      lane, a.x, a.y, bx, by);
                if (__any(far)) {
                    big_sym_block<true>(C, &L.tab, own, own.fx, own.fy, L.src[w], s_lo, s_full, s_hi, lane, a.x, a.y,
                                        cx, cy);
                    bx += cx;
                    by += cy;
                }
                if (m) *m = V2<double>{bx, by};
            };
            if (k == A) {
                // the diagonal block: offsets 1..32, offset 32 for lanes 0..31
                V2<double> t{0.0, 0.0};
                target(1, 32, 33, t, &P);
                L.diag[lane] = t;
            } else if (k > A) {
                target(0, 64, 64, P, nullptr);
            } else {
                double ax = 0.0, ay = 0.0, cx, cy;
                const bool far = big_sym_block<false>(C, &L.tab, q, q.fx, q.fy, L.own, 0, 64, 64, lane, ax, ay, P.x, P.y);
                if (__any(far)) {
                    big_sym_block<true>(C, &L.tab, q, q.fx, q.fy, L.own, 0, 64, 64, lane, ax, ay, cx, cy);
                    P.x += cx;
                    P.y += cy;
                }
            }
        }
        L.part[w][lane] = P;
        __syncthreads();
        if (w == 0) {
            for (int j = 0; j < VEL_WAVES && k0 + j < 2 * nt; j += 2) {
                const V2<double> e = L.part[j][lane], f = L.part[j + 1][lane];
                if (k0 + j != 2 * tA) {
                    u += e.x + f.x;
                    v += e.y + f.y;
                } else {
                    // the own tile: moving sums by block, then target sums
                    const V2<double> t = L.diag[lane];
                    u += A & 1 ? (e.x + f.x) + t.x : e.x + (t.x + f.x);
                    v += A & 1 ? (e.y + f.y) + t.y : e.y + (t.y + f.y);
                }
            }
        }
    }
    const int i = 64 * A + lane;
    if (w != 0 || i >= n) return;
    const double h1c = C.h1c;
    ux[p0 + i] = (float)fma(h1c, L.red[0][0] + L.red[0][1] + L.red[0][2] + L.red[0][3], u);
    uy[p0 + i] = (float)fma(h1c, L.red[1][0] + L.red[1][1] + L.red[1][2] + L.red[1][3], v);
}

// sources (position, force at t = 0) of the large systems' first step
__global__ __launch_bounds__(256) void k_big_sources(BigTiles bt, Batch b, BigState S)
{
    const int64_t g = blockIdx.y, s = bt.list[g], p0 = bt.pt0[g];
    const int n = bt.cnt[g];
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256)
        reinterpret_cast<Src4<float>*>(bt.src)[p0 + i] =
            big_source<float>(b, (const float*)S.xh[0] + p0, (const float*)S.yh[0] + p0, (const float*)S.xl[0] + p0,
                              (const float*)S.yl[0] + p0, b.sw_off[s], b.npt[s], i, 0.0f);
}

// The Euler step of the tile-pair path, one workgroup per tile: a point's
// velocity is the sum of its tile's slots in tile order (SG groups of threads
// each a share of the slots, added in order), then the new positions of the
// tile and of two points on either side, and from them the elastic forces of
// the tile's points at the new time: the sources of the next step, formed
// once per point instead of by every tile pair that reads them.
constexpr int BIG_HALO = 2, UPD_PT = (BT + 2 * BIG_HALO + 63) / 64 * 64, UPD_SG = 4;
__global__ __launch_bounds__(UPD_PT* UPD_SG) void k_big_update(BigTiles bt, Batch b, BigState S, int step, Run r,
                                                               float* obs, int32_t* status, int32_t* steps_done)
{
    constexpr int PT = UPD_PT, SG = UPD_SG;
    __shared__ V2<double> sum[SG][PT];
    __shared__ float4 pos[PT];  // hi x, hi y, lo x, lo y
    __shared__ int s_status;
    const int tid = threadIdx.x % PT, sg = threadIdx.x / PT;
    const int64_t g = prefix_item(bt.tile0, bt.n_big, blockIdx.x);
    const int tile = (int)((int64_t)blockIdx.x - bt.tile0[g]);
    const int64_t s = bt.list[g];
    if (threadIdx.x == 0) s_status = status[s];
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_status) != 0) return;
    const int64_t p0 = bt.pt0[g];
    const int N = b.npt[s], n = bt.cnt[g], nt = (n + BT - 1) / BT;
    const int64_t f0 = b.sw_off[s];
    const int cur = step & 1, nxt = cur ^ 1;
    const int i = tile * BT + tid - BIG_HALO;  // this thread's point (halo points belong to the next tiles)
    const bool held = tid < BT + 2 * BIG_HALO && i >= 0 && i < n;
    const bool own = held && tid >= BIG_HALO && tid < BT + BIG_HALO;
    double ux = 0.0, uy = 0.0;
    if (held) {
        const int t = i / BT, per = (nt + SG - 1) / SG, q1 = min(nt, (sg + 1) * per);
        const V2<double>* src =
            reinterpret_cast<const V2<double>*>(bt.part) + (bt.slot0[g] + (int64_t)t * nt) * BT + (i - t * BT);
#pragma unroll 4
        for (int q = sg * per; q < q1; ++q) {
            const V2<double> v = src[(int64_t)q * BT];
            ux += v.x;
            uy += v.y;
        }
    }
    sum[sg][tid] = V2<double>{ux, uy};
    __syncthreads();
    if (sg == 0 && held) {
#pragma unroll
        for (int k = 1; k < SG; ++k) {
            ux += sum[k][tid].x;
            uy += sum[k][tid].y;
        }
        float hx = ((const float*)S.xh[cur])[p0 + i], hy = ((const float*)S.yh[cur])[p0 + i];
        float lx = ((const float*)S.xl[cur])[p0 + i], ly = ((const float*)S.yl[cur])[p0 + i];
        const float dt = (float)r.dt;
        if (own)
            big_update_point<float>(S, step, r, s, p0, f0, N, i, nxt, hx, hy, lx, ly, (float)ux, (float)uy, obs,
                                    status, steps_done);
        acc2(hx, lx, dt * (float)ux);
        acc2(hy, ly, dt * (float)uy);
        pos[tid] = make_float4(hx, hy, lx, ly);
    }
    __syncthreads();
    const int j = tile * BT + (int)threadIdx.x;
    if ((int)threadIdx.x < BT && j < n) {
        const int m = j / N, p = j - m * N, base = m * N - (tile * BT - BIG_HALO);
        const FilP<float> q = load_filp<float>(b.params, f0 + m, N);
        auto seg = [&](int k, float& dx, float& dy) {
            const float4 e = pos[base + k], f = pos[base + k + 1];
            dx = (f.x - e.x) + (f.z - e.z);
            dy = (f.y - e.y) + (f.w - e.w);
        };
        Src4<float> v;
        point_force<float>(seg, p, q, (float)((double)(step + 1) * r.dt), v.fx, v.fy);
        v.x = pos[threadIdx.x + BIG_HALO].x;
        v.y = pos[threadIdx.x + BIG_HALO].y;
        reinterpret_cast<Src4<float>*>(bt.src)[p0 + j] = v;
    }
}

template <typename T>
__global__ void k_big_finish(const int64_t* list, Batch b, BigState S, int buf, Run r, T* speed,
                             const int32_t* status, int32_t* steps_done)
{
    const int64_t s = list[blockIdx.x];
    if (threadIdx.x == 0 && steps_done) {
        if (status[s] == 0) steps_done[s] = r.steps;
        else if (status[s] == SWIM_ST_BADPARAM_) steps_done[s] = 0;
    }
    const int64_t p0 = b.pt_off[s];
    const int N = b.npt[s];
    const int nsw = b.nswim[s];
    const T Tend = (T)((double)r.steps * r.dt);
    for (int m = threadIdx.x; m < nsw; m += blockDim.x) {
        const int64_t f = b.sw_off[s] + m;
        const int64_t i = p0 + (int64_t)m * N + N - 1;
        if (status[s]) {
            speed[f] = (T)NAN;
        } else {
            const T hx = ((const T*)S.xh[buf])[i] + ((const T*)S.xl[buf])[i];
            const T hy = ((const T*)S.yh[buf])[i] + ((const T*)S.yl[buf])[i];
            const T dx = hx - ((const T*)S.head0)[2 * f], dy = hy - ((const T*)S.head0)[2 * f + 1];
            speed[f] = sqrt_t(fma_t(dx, dx, dy * dy)) / Tend;
        }
    }
}

// ---------------------------------------------------------------------------
// ABC: RMS head-position distance, k-th smallest (radix select), accept mask
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_abc_distance(int64_t n, int32_t n_obs, const T* obs, const double* data, const int32_t* status,
                               double* dist)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const T* o = obs + i * (int64_t)n_obs * 2;
    double acc = 0.0;
    for (int m = 0; m < 2 * n_obs; ++m) {
        const double d = (double)o[m] - data[m];
        acc = fma(d, d, acc);
    }
    double d = sqrt(acc / (2.0 * n_obs));
    if ((status && status[i] != 0) || !isfinite(d)) d = INFINITY;
    dist[i] = d;
}

__device__ __forceinline__ uint64_t dkey(double v)
{
    const uint64_t u = __double_as_longlong(v);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double dunkey(uint64_t k)
{
    const uint64_t u = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __longlong_as_double(u);
}

// tolerance = k-th smallest finite value of v, k = ceil(q * n_finite)
// clamped to [1, n_finite] (+inf when no value is finite): count the finite
// values, then an 8-pass MSB-first radix select over the order-preserving
// 64-bit keys of the doubles.  One workgroup.
__global__ __launch_bounds__(1024) void k_select_kth(int64_t n, const double* v, double q, double* out)
{
    __shared__ unsigned int hist[256];
    __shared__ uint64_t s_prefix, s_mask;
    __shared__ int64_t s_rank;
    __shared__ unsigned long long s_nf;
    const int tid = threadIdx.x;
    if (tid == 0) s_nf = 0;
    __syncthreads();
    unsigned long long nf = 0;
    for (int64_t i = tid; i < n; i += blockDim.x) nf += isfinite(v[i]) ? 1 : 0;
    atomicAdd(&s_nf, nf);
    __syncthreads();
    const int64_t n_fin = (int64_t)s_nf;
    if (n_fin == 0) {
        if (tid == 0) *out = INFINITY;
        return;
    }
    if (tid == 0) {
        int64_t k = (int64_t)ceil(q * (double)n_fin);
        k = k < 1 ? 1 : (k > n_fin ? n_fin : k);
        s_prefix = 0;
        s_mask = 0;
        s_rank = k - 1;
    }
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
        for (int h = tid; h < 256; h += blockDim.x) hist[h] = 0;
        __syncthreads();
        const uint64_t prefix = s_prefix, mask = s_mask;
        for (int64_t i = tid; i < n; i += blockDim.x) {
            const uint64_t key = dkey(v[i]);
            if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid == 0) {
            int64_t r = s_rank, cum = 0;
            int d = 0;
            for (; d < 256; ++d) {
                if (r < cum + (int64_t)hist[d]) break;
                cum += hist[d];
            }
            s_rank = r - cum;
            s_prefix = prefix | ((uint64_t)d << shift);
            s_mask = mask | ((uint64_t)255 << shift);
        }
        __syncthreads();
    }
    if (tid == 0) *out = dunkey(s_prefix);
}

__global__ void k_accept(int64_t n, const double* dist, const double* tol, uint8_t* acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) acc[i] = (isfinite(dist[i]) && dist[i] <= *tol) ? 1 : 0;
}

// Gaussian log-likelihood of each forward run (eqs. likelihood, fitness with
// Sigma = sigma_i^2 I over the m = 2 n_obs head coordinates, in the order
// x_0, y_0, x_1, y_1, ...): -m/2 log(2 pi) - m log(sigma_i) - J/2 with
// J = |D - g|^2 / sigma_i^2, in FP64; -inf for a run that did not complete.
template <typename T>
__global__ void k_gauss_loglik(int64_t n, int32_t n_obs, const T* obs, const double* data, const double* sigma,
                               const int32_t* status, double* logl)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (status[i] != 0) {
        logl[i] = -INFINITY;
        return;
    }
    const T* g = obs + i * (int64_t)n_obs * 2;
    double J = 0.0;
    for (int k = 0; k < 2 * n_obs; ++k) {
        const double r = data[k] - (double)g[k];
        J = fma(r, r, J);
    }
    const double sg = sigma[i], m = 2.0 * n_obs;
    logl[i] = -0.5 * m * log(2.0 * M_PI) - m * log(sg) - 0.5 * J / (sg * sg);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

hipError_t launch_sysconst_batch(int dtype, int64_t n_sys, const int64_t* sw_off, const int32_t* npt,
                                 const double* params, double eps_over_ds, void* sysc, void* sysc64,
                                 int32_t* status, int blob, hipStream_t st)
{
    if (n_sys <= 0) return hipSuccess;
    if (!grid_fits(n_sys, 64)) return hipErrorInvalidConfiguration;
    if (dtype == 0)
        hipLaunchKernelGGL(k_sysconst_batch<float>, dim3((unsigned)n_sys), dim3(64), 0, st, sw_off, npt, params,
                           eps_over_ds, (SysConst<float>*)sysc, (SysConst<double>*)sysc64, status, blob);
    else
        hipLaunchKernelGGL(k_sysconst_batch<double>, dim3((unsigned)n_sys), dim3(64), 0, st, sw_off, npt, params,
                           eps_over_ds, (SysConst<double>*)sysc, (SysConst<double>*)nullptr, status, blob);
    return hipGetLastError();
}

hipError_t launch_sysconst(int dtype, int64_t n_sys, const double* alpha, const double* eps, void* sysc,
                           void* sysc64, int blob, hipStream_t st)
{
    if (n_sys <= 0) return hipSuccess;
    if (!grid_fits(n_sys, 64)) return hipErrorInvalidConfiguration;
    if (dtype == 0)
        hipLaunchKernelGGL(k_sysconst<float>, dim3((unsigned)n_sys), dim3(64), 0, st, alpha, eps,
                           (SysConst<float>*)sysc, (SysConst<double>*)sysc64, blob);
    else
        hipLaunchKernelGGL(k_sysconst<double>, dim3((unsigned)n_sys), dim3(64), 0, st, alpha, eps,
                           (SysConst<double>*)sysc, (SysConst<double>*)nullptr, blob);
    return hipGetLastError();
}

size_t table_bytes(int dtype) { return dtype == 0 ? sizeof(TabSys) : sizeof(TabSys64); }

hipError_t launch_table_build(int dtype, int64_t s0, int64_t n, const void* sysc64, void* tab, int blob, hipStream_t st,
                              const int64_t* pt_off)
{
    if (n <= 0) return hipSuccess;
    if (!grid_fits(n, PB_BLOCK) || !grid_fits(n * TAB_WAVES, 64)) return hipErrorInvalidConfiguration;
    if (dtype == 1)
        hipLaunchKernelGGL(k_table_build_pb<9>, dim3((unsigned)n), dim3(PB_BLOCK), 0, st, s0,
                           (const SysConst<double>*)sysc64, tab, pt_off);
    else if (blob == 1)
        hipLaunchKernelGGL(k_table_build_pb<7>, dim3((unsigned)n), dim3(PB_BLOCK), 0, st, s0,
                           (const SysConst<double>*)sysc64, tab, (const int64_t*)nullptr);
    else
        hipLaunchKernelGGL(k_table_build, dim3((unsigned)(n * TAB_WAVES)), dim3(64), 0, st, s0, n,
                           (const SysConst<double>*)sysc64, (TabSys*)tab);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(nblk(n, 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

hipError_t launch_pair_velocity(int dtype, int64_t n_sys, int64_t nb, const int64_t* blk0, const int64_t* off,
                                const void* sysc, const void* tab, const void* x, const void* y, const void* fx,
                                const void* fy, void* ux, void* uy, hipStream_t st)
{
    if (nb <= 0) return hipSuccess;
    if (!grid_fits(nb, 64 * VEL_WAVES)) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)nb), block(64 * VEL_WAVES);
    if (dtype == 0)
        hipLaunchKernelGGL(k_pair_velocity<float>, grid, block, 0, st, n_sys, blk0, off, (const SysConst<float>*)sysc,
                           tab, (const float*)x, (const float*)y, (const float*)fx, (const float*)fy, (float*)ux,
                           (float*)uy);
    else
        hipLaunchKernelGGL(k_pair_velocity<double>, grid, block, 0, st, n_sys, blk0, off,
                           (const SysConst<double>*)sysc, tab, (const double*)x, (const double*)y, (const double*)fx,
                           (const double*)fy, (double*)ux, (double*)uy);
    return hipGetLastError();
}

hipError_t launch_direct_velocity(int64_t n_sys, int64_t nb, const int64_t* blk0, const int64_t* off, const void* sysc,
                                  const void* x, const void* y, const void* fx, const void* fy, void* ux, void* uy,
                                  hipStream_t st)
{
    if (nb <= 0) return hipSuccess;
    if (!grid_fits(nb, 64)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_direct_velocity, dim3((unsigned)nb), dim3(64), 0, st, n_sys, blk0, off,
                       (const SysConst<double>*)sysc, (const double*)x, (const double*)y, (const double*)fx,
                       (const double*)fy, (double*)ux, (double*)uy);
    return hipGetLastError();
}

hipError_t launch_ordered_velocity(int64_t n_sys, int64_t nb, const int64_t* blk0, const int64_t* off, const void* sysc,
                                   const void* tab, const void* x, const void* y, const void* fx, const void* fy,
                                   void* ux, void* uy, hipStream_t st)
{
    if (nb <= 0) return hipSuccess;
    if (!grid_fits(nb, 64 * VEL_WAVES)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_ordered_velocity, dim3((unsigned)nb), dim3(64 * VEL_WAVES), 0, st, n_sys, blk0, off,
                       (const SysConst<float>*)sysc, (const TabSys*)tab, (const float*)x, (const float*)y,
                       (const float*)fx, (const float*)fy, (float*)ux, (float*)uy);
    return hipGetLastError();
}

template <bool SOA>
static hipError_t tile_prepare()
{
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void*)k_tile_pairs<SOA>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)TileLds::total);
        if (e != hipSuccess) return e;
        attr = true;
    }
    return hipSuccess;
}

hipError_t launch_tile_velocity(const BigTiles& bt, const void* sysc, const void* tab, const void* x, const void* y,
                                const void* fx, const void* fy, void* ux, void* uy, hipStream_t st)
{
    if (bt.n_big <= 0) return hipSuccess;
    if (!grid_fits(bt.n_pairs, 256) || !grid_fits(bt.n_tiles, 256)) return hipErrorInvalidConfiguration;
    hipError_t e = tile_prepare<true>();
    if (e != hipSuccess) return e;
    const SysConst<float>* C = (const SysConst<float>*)sysc;
    hipLaunchKernelGGL(k_tile_pairs<true>, dim3((unsigned)bt.n_pairs), dim3(256), TileLds::total, st, bt, C,
                       (const TabSys*)tab, (const float*)x, (const float*)y, (const float*)fx, (const float*)fy,
                       (const int32_t*)nullptr);
    hipLaunchKernelGGL(k_tile_velocity, dim3((unsigned)bt.n_tiles), dim3(256), 0, st, bt, C, (const float*)fx,
                       (const float*)fy, (float*)ux, (float*)uy);
    return hipGetLastError();
}

hipError_t launch_forces(int dtype, int64_t n_fil, const int64_t* fil_off, const int32_t* npt, const double* params,
                         double t, const void* x, const void* y, void* fx, void* fy, hipStream_t st)
{
    if (n_fil <= 0) return hipSuccess;
    // grid.y covers filaments; grid.x covers up to 4096 points per filament
    const dim3 grid(16, (unsigned)n_fil);
    if (dtype == 0)
        hipLaunchKernelGGL(k_forces<float>, grid, dim3(256), 0, st, n_fil, fil_off, npt, params, t, (const float*)x,
                           (const float*)y, (float*)fx, (float*)fy);
    else
        hipLaunchKernelGGL(k_forces<double>, grid, dim3(256), 0, st, n_fil, fil_off, npt, params, t,
                           (const double*)x, (const double*)y, (double*)fx, (double*)fy);
    return hipGetLastError();
}

hipError_t launch_order_runs(int n_seg, const OrderSegs& seg, const int32_t* in, const int64_t* sw_off,
                             const int32_t* npt, const double* params, double dt, int32_t* out, hipStream_t st)
{
    if (n_seg <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_order_runs, dim3((unsigned)n_seg), dim3(1024), 0, st, seg, in, sw_off, npt, params, dt, out);
    return hipGetLastError();
}

size_t forward_lds_bytes(int dtype, int tpl, int wps) { return fwd_lds_layout(dtype, tpl, wps).total; }

// shapes with a second build: FP32 reading ahead, FP64 with the table in LDS
template <typename T> constexpr bool fwd_second_build(int tpl, int wps)
{
    return sizeof(T) == 4 ? tpl <= 2 && fwd_window(0, tpl, wps) : fwd_lds64(1, tpl, wps);
}

// raise the kernel's dynamic-LDS limit to what its launches need (outside
// any stream capture: a launch inside a capture finds it already set)
template <typename T, int TPL, int WPS>
static hipError_t fwd_prepare()
{
    const size_t lds = forward_lds_bytes(sizeof(T) == 4 ? 0 : 1, TPL, WPS);
    static size_t attr_lds = 0;
    if (lds > attr_lds) {
        hipError_t e = hipFuncSetAttribute((const void*)k_forward<T, TPL, WPS>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if constexpr (fwd_second_build<T>(TPL, WPS)) {
            if (e == hipSuccess)
                e = hipFuncSetAttribute((const void*)k_forward<T, TPL, WPS, true>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)fwd_lds_layout(sizeof(T) == 4 ? 0 : 1, TPL, WPS, sizeof(T) == 8).total);
        }
        if (e != hipSuccess) return e;
        attr_lds = lds;
    }
    return hipSuccess;
}

template <typename T, int TPL, int WPS>
static hipError_t fwd_launch(int nblocks, const Batch& b, const Run& r, const int32_t* order, int32_t* q, void* obs,
                             void* speed, int32_t* status, int32_t* done, hipStream_t st)
{
    const size_t lds = forward_lds_bytes(sizeof(T) == 4 ? 0 : 1, TPL, WPS);
    hipError_t e = fwd_prepare<T, TPL, WPS>();
    if (e != hipSuccess) return e;
    if constexpr (fwd_second_build<T>(TPL, WPS)) {
        if (sizeof(T) == 4 ? b.alone != 0 : r.steps >= FWD_LDS64_STEPS) {
            const size_t own = fwd_lds_layout(sizeof(T) == 4 ? 0 : 1, TPL, WPS, sizeof(T) == 8).total;
            hipLaunchKernelGGL((k_forward<T, TPL, WPS, true>), dim3(nblocks), dim3(64 * WPS), own, st, b, r, order, q,
                               (T*)obs, (T*)speed, status, done);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_forward<T, TPL, WPS>), dim3(nblocks), dim3(64 * WPS), lds, st, b, r, order, q, (T*)obs,
                       (T*)speed, status, done);
    return hipGetLastError();
}

template <typename T, int TPL, int WPS>
static int fwd_occupancy()
{
    int nb = 0;
    const size_t lds = forward_lds_bytes(sizeof(T) == 4 ? 0 : 1, TPL, WPS);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_forward<T, TPL, WPS>, 64 * WPS, lds) != hipSuccess || nb < 1)
        nb = 1;
    return nb;
}

// instantiated launch shapes (targets per lane, waves per system): every
// wave count from forward_min_wps(tpl) up
#define SWIM_FWD_TABLE(X, T)                                                                               \
    X(T, 1, 1) X(T, 1, 2) X(T, 1, 4) X(T, 1, 8) X(T, 1, 16) X(T, 2, 1) X(T, 2, 2) X(T, 2, 4) X(T, 2, 8)      \
    X(T, 2, 16) X(T, 3, 1) X(T, 3, 2) X(T, 3, 4) X(T, 3, 8) X(T, 3, 16) X(T, 4, 1) X(T, 4, 2) X(T, 4, 4)     \
    X(T, 4, 8) X(T, 4, 16) X(T, 6, 2) X(T, 6, 4) X(T, 6, 8) X(T, 6, 16) X(T, 8, 2) X(T, 8, 4) X(T, 8, 8)      \
    X(T, 8, 16)

int forward_min_wps(int tpl)
{
    const int nwin = (64 * tpl + FWD_WIN - 1) / FWD_WIN;
    int w = 1;
    while ((nwin + w - 1) / w > FWD_MAX_WINDOWS) w *= 2;
    return w;
}

hipError_t launch_forward(int dtype, int tpl, int wps, int nblocks, const Batch& b, const Run& r,
                          const int32_t* order, int32_t* queue, void* obs, void* speed, int32_t* status,
                          int32_t* steps_done, hipStream_t st)
{
#define FWD_CASE(T, P, W) \
    if (tpl == P && wps == W) return fwd_launch<T, P, W>(nblocks, b, r, order, queue, obs, speed, status, steps_done, st);
    if (dtype == 0) {
        SWIM_FWD_TABLE(FWD_CASE, float)
    } else {
        SWIM_FWD_TABLE(FWD_CASE, double)
    }
#undef FWD_CASE
    return hipErrorInvalidValue;
}

hipError_t prepare_forward(int dtype, int tpl, int wps)
{
#define PREP_CASE(T, P, W) \
    if (tpl == P && wps == W) return fwd_prepare<T, P, W>();
    if (dtype == 0) {
        SWIM_FWD_TABLE(PREP_CASE, float)
    } else {
        SWIM_FWD_TABLE(PREP_CASE, double)
    }
#undef PREP_CASE
    return hipErrorInvalidValue;
}

int forward_blocks_per_cu(int dtype, int tpl, int wps)
{
#define OCC_CASE(T, P, W) \
    if (tpl == P && wps == W) return fwd_occupancy<T, P, W>();
    if (dtype == 0) {
        SWIM_FWD_TABLE(OCC_CASE, float)
    } else {
        SWIM_FWD_TABLE(OCC_CASE, double)
    }
#undef OCC_CASE
    return 1;
}

hipError_t launch_big_init(int dtype, const int64_t* list, int64_t n_list, const Batch& b, const BigState& s,
                           int32_t* status, void* obs, int32_t n_obs, hipStream_t st)
{
    if (n_list <= 0) return hipSuccess;
    const dim3 grid(16, (unsigned)n_list);
    if (dtype == 0)
        hipLaunchKernelGGL(k_big_init<float>, grid, dim3(256), 0, st, list, b, s, status, (float*)obs, n_obs);
    else
        hipLaunchKernelGGL(k_big_init<double>, grid, dim3(256), 0, st, list, b, s, status, (double*)obs, n_obs);
    return hipGetLastError();
}

size_t big_step_lds_bytes(int dtype, int32_t max_pts)
{
    (void)max_pts;  // sources are tiled: any system size
    return (dtype == 0 ? table_bytes(0) : 0) + (size_t)BIG_TILE * 4 * (dtype == 0 ? sizeof(float) : sizeof(double));
}

template <typename T, int TPL>
static hipError_t big_prepare(int32_t max_pts)
{
    const size_t lds = big_step_lds_bytes(sizeof(T) == 4 ? 0 : 1, max_pts);
    static size_t attr_lds = 0;
    if (lds > attr_lds) {
        hipError_t e = hipFuncSetAttribute((const void*)k_big_step<T, TPL>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_lds = lds;
    }
    return hipSuccess;
}

hipError_t prepare_big_step(int dtype, int tpl, int32_t max_pts)
{
    if (dtype == 0) {
        switch (tpl) {
            case 1: return big_prepare<float, 1>(max_pts);
            case 2: return big_prepare<float, 2>(max_pts);
            case 4: return big_prepare<float, 4>(max_pts);
            default: return hipErrorInvalidValue;
        }
    }
    switch (tpl) {
        case 1: return big_prepare<double, 1>(max_pts);
        case 2: return big_prepare<double, 2>(max_pts);
        case 4: return big_prepare<double, 4>(max_pts);
        default: return hipErrorInvalidValue;
    }
}

template <typename T, int TPL>
static hipError_t big_launch(int64_t nb, const int64_t* bs, const int64_t* bf, int32_t max_pts, const Batch& b,
                             const BigState& s, int step, const Run& r, void* obs, int32_t* status, int32_t* done,
                             hipStream_t st)
{
    const size_t lds = big_step_lds_bytes(sizeof(T) == 4 ? 0 : 1, max_pts);
    hipError_t e = big_prepare<T, TPL>(max_pts);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_big_step<T, TPL>), dim3((unsigned)nb), dim3(256), lds, st, bs, bf, b, s, step, r, (T*)obs,
                       status, done);
    return hipGetLastError();
}

hipError_t launch_big_step(int dtype, int tpl, int64_t nb, const int64_t* bs, const int64_t* bf, int32_t max_pts,
                           const Batch& b, const BigState& s, int step, const Run& r, void* obs, int32_t* status,
                           int32_t* steps_done, hipStream_t st)
{
#define BIG_CASE(T, P) \
    case P: return big_launch<T, P>(nb, bs, bf, max_pts, b, s, step, r, obs, status, steps_done, st);
    if (dtype == 0) {
        switch (tpl) { BIG_CASE(float, 1) BIG_CASE(float, 2) BIG_CASE(float, 4) default: return hipErrorInvalidValue; }
    } else {
        switch (tpl) { BIG_CASE(double, 1) BIG_CASE(double, 2) BIG_CASE(double, 4) default: return hipErrorInvalidValue; }
    }
#undef BIG_CASE
}

// raise k_tile_pairs' dynamic-LDS limit (outside any stream capture)
hipError_t prepare_big_pairs() { return tile_prepare<false>(); }

hipError_t launch_big_sources(const BigTiles& bt, const Batch& b, const BigState& s, hipStream_t st)
{
    if (bt.n_big <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_big_sources, dim3(16, (unsigned)bt.n_big), dim3(256), 0, st, bt, b, s);
    return hipGetLastError();
}

hipError_t launch_big_sym_step(const BigTiles& bt, const Batch& b, const BigState& s, int step, const Run& r, void* obs,
                               int32_t* status, int32_t* steps_done, hipStream_t st)
{
    if (bt.n_big <= 0) return hipSuccess;
    if (!grid_fits(bt.n_pairs, 256) || !grid_fits(bt.n_tiles, UPD_PT * UPD_SG)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_tile_pairs<false>, dim3((unsigned)bt.n_pairs), dim3(256), TileLds::total, st, bt,
                       (const SysConst<float>*)b.sysc, (const TabSys*)b.tab, (const float*)nullptr,
                       (const float*)nullptr, (const float*)nullptr, (const float*)nullptr, (const int32_t*)status);
    hipLaunchKernelGGL(k_big_update, dim3((unsigned)bt.n_tiles), dim3(UPD_PT * UPD_SG), 0, st, bt, b, s, step, r,
                       (float*)obs, status, steps_done);
    return hipGetLastError();
}

hipError_t launch_big_finish(int dtype, const int64_t* list, int64_t n_list, const Batch& b, const BigState& s,
                             int buf, const Run& r, void* speed, const int32_t* status, int32_t* steps_done,
                             hipStream_t st)
{
    if (n_list <= 0) return hipSuccess;
    if (dtype == 0)
        hipLaunchKernelGGL(k_big_finish<float>, dim3((unsigned)n_list), dim3(64), 0, st, list, b, s, buf, r,
                           (float*)speed, status, steps_done);
    else
        hipLaunchKernelGGL(k_big_finish<double>, dim3((unsigned)n_list), dim3(64), 0, st, list, b, s, buf, r,
                           (double*)speed, status, steps_done);
    return hipGetLastError();
}

hipError_t launch_abc_distance(int dtype, int64_t n, int32_t n_obs, const void* obs, const double* data,
                               const int32_t* status, double* dist, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (dtype == 0)
        hipLaunchKernelGGL(k_abc_distance<float>, dim3(nblk(n, 256)), dim3(256), 0, st, n, n_obs, (const float*)obs,
                           data, status, dist);
    else
        hipLaunchKernelGGL(k_abc_distance<double>, dim3(nblk(n, 256)), dim3(256), 0, st, n, n_obs,
                           (const double*)obs, data, status, dist);
    return hipGetLastError();
}

hipError_t launch_select_kth(int64_t n, const double* v, double q, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_select_kth, dim3(1), dim3(1024), 0, st, n, v, q, out);
    return hipGetLastError();
}

hipError_t launch_accept(int64_t n, const double* dist, const double* tol, uint8_t* acc, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_accept, dim3(nblk(n, 256)), dim3(256), 0, st, n, dist, tol, acc);
    return hipGetLastError();
}

hipError_t launch_gauss_loglik(int dtype, int64_t n, int32_t n_obs, const void* obs, const double* data,
                               const double* sigma, const int32_t* status, double* logl, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (dtype == 0)
        hipLaunchKernelGGL(k_gauss_loglik<float>, dim3(nblk(n, 256)), dim3(256), 0, st, n, n_obs, (const float*)obs,
                           data, sigma, status, logl);
    else
        hipLaunchKernelGGL(k_gauss_loglik<double>, dim3(nblk(n, 256)), dim3(256), 0, st, n, n_obs, (const double*)obs,
                           data, sigma, status, logl);
    return hipGetLastError();
}

}  // namespace swim

