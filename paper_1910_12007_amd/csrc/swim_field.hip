// swim_field.hip -- velocity (eq. BrV) and pressure (eq. BrP) of the
// regularized point forces of one system at arbitrary target points (Sec.
// 2.1), for flow and pressure pictures of a swimmer.
//
// Pressure: p = sum_i F_i . grad G_eps(x - X_i) with Delta G_eps = phi, the
// blob of the velocity kernel.  For a radial blob grad G_eps(x) =
// x m(r) / (2 pi r^2), m(r) the blob mass inside r; from (Delta - alpha^2) g
// = phi, m/(2 pi) = r g' - alpha^2 M, so for this blob
//   Stokes:   m = r^2 / R^2,
//   Brinkman: m = 1 - eps K1(alpha R) / (R K1(alpha eps)),  R^2 = r^2 + eps^2,
// and near contact (delta = r^2/eps^2 < 1/4) w = m / (2 pi r^2) is a power
// series in delta whose coefficients the host computes per call.
//
// One thread per target; the sources pass through LDS in tiles; every sum is
// accumulated in FP64.  The pair kernel comes from the system's table, as in
// the forward runs.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "swim_internal.h"
#include "swim_math.h"
#include "swim_pairsum.h"

namespace swim {

namespace {

constexpr int FIELD_TILE = 256;  // sources per LDS tile, threads per workgroup

// pressure weight m(r) / (2 pi r^2) at t = r^2, in FP64
__device__ double field_weight(const FieldConst& fc, double t)
{
    const double delta = t * fc.inv_e2;
    if (fc.paper) {
        // m = 1 - eps^3/R^3:  w = (R^2 + R eps + eps^2) / (2 pi R^3 (R + eps))
        const double R2 = t + fc.e2, R = sqrt(R2);
        return fc.inv_2pi * (R2 + R * fc.eps + fc.e2) / (R2 * R * (R + fc.eps));
    }
    if (fc.stokes) return fc.inv_2pi / (t + fc.e2);
    if (delta < 0.25) {
        double w = fc.ser[FIELD_NSER - 1];
        for (int q = FIELD_NSER - 2; q >= 0; --q) w = fma(w, delta, fc.ser[q]);
        return w;
    }
    const double R = sqrt(t + fc.e2);
    double K0, K1, Q;
    bessel_k01_q_f64(fc.alpha * R, &K0, &K1, &Q);
    return fc.inv_2pi * (1.0 - fc.eps * K1 / (R * fc.K1e)) / t;
}

// FP32 table of the pressure weight on the kernel table's intervals of
// v = 1 + sigma t: the cubic through its FP64 values at the nodes 0, 1/4,
// 3/4, 1 of each interval (one thread per interval), then a zero entry
__global__ __launch_bounds__(256) void k_weight_table(const FieldConst* fcp, float4* wt)
{
    const FieldConst& fc = *fcp;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i > TAB_N) return;
    if (i == TAB_N) {
        wt[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        return;
    }
    const int e = i >> TAB_M, j = i & ((1 << TAB_M) - 1);
    const double a = ldexp(1.0, e);
    const double v0 = a * (1.0 + (double)j / (double)(1 << TAB_M)), hv = a / (double)(1 << TAB_M);
    const double un[4] = {0.0, 0.25, 0.75, 1.0};
    double f[4];
    for (int k = 0; k < 4; ++k) f[k] = field_weight(fc, fmax((v0 - 1.0 + hv * un[k]) * fc.c64.its, 1e-300));
    float c[4];
    cubic_lobatto(f, ldexp(1.0, -TAB_SHIFT), 1.0, c);
    wt[i] = make_float4(c[0], c[1], c[2], c[3]);
}

// FP32 values of a pair beyond the tables (or not finite), evaluated directly;
// not inlined, so that its registers stay out of the pair loop
struct FieldFar {
    float Ht, H2;
    double w;
};
__device__ __attribute__((noinline)) FieldFar field_far(const FieldConst& fc, float t2, double t)
{
    FieldFar f;
    kernel_eval<float>(fc.c32, t2, f.Ht, f.H2);
    f.w = field_weight(fc, t);
    return f;
}
// one interval of the two FP32 tables together: Ht, H2 / sigma and the
// pressure weight, three 16-byte reads at one address
struct alignas(16) FieldE {
    float4 h, g, w;
};
// a source in both precisions (position times rho in FP32)
struct alignas(16) FieldSrc {
    double x, y, fx, fy;
    float4 f;
};

// FP32 fields, TPL targets per thread.  The kernel table and the pressure
// weight's are merged in LDS (34 KB); sources pass through LDS in both
// precisions, so that a pair costs the FP64 difference (for the pressure),
// the FP32 table lookup on scaled positions, three cubics and three FP64
// accumulations: ~40 operations, bound by VALU issue.  Neighbouring targets
// read the same few entries.  A picture of 1024 x 1024 targets and 256
// sources took 727 us with the tables gathered from L1, positions converted
// and the forces summed again by every thread.  Two targets per thread share
// a source's reads where the picture fills the chip anyway.
template <int TPL>
__global__ __launch_bounds__(FIELD_TILE) void k_flow_field32(int64_t n, const float* x, const float* y,
                                                             const float* fx, const float* fy, const FieldConst* fcp,
                                                             int64_t nt, const float* tx, const float* ty, float* u,
                                                             float* v, float* p, const TabSys* tab, const float4* wtab)
{
    __shared__ FieldE tb[TAB_N + 1];
    __shared__ FieldSrc tile[FIELD_TILE];
    __shared__ double red[2][FIELD_TILE / 64];
    const FieldConst& fc = *fcp;
    const int tid = threadIdx.x;
    for (int i = tid; i <= TAB_N; i += FIELD_TILE) {
        const float4* e = reinterpret_cast<const float4*>(&tab->e[i]);
        tb[i] = FieldE{e[0], e[1], wtab[i]};
    }
    const float rho = fc.c32.tr;
    int64_t a[TPL];
    double X[TPL], Y[TPL], su[TPL], sv[TPL], sp[TPL];
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
        a[q] = ((int64_t)blockIdx.x * TPL + q) * FIELD_TILE + tid;
        X[q] = a[q] < nt ? (double)tx[a[q]] : 0.0;
        Y[q] = a[q] < nt ? (double)ty[a[q]] : 0.0;
        su[q] = sv[q] = sp[q] = 0.0;
    }
    double sfx = 0.0, sfy = 0.0;
    for (int64_t j0 = 0; j0 < n; j0 += FIELD_TILE) {
        const int m = (int)min<int64_t>(FIELD_TILE, n - j0);
        __syncthreads();
        if (tid < m) {
            const int64_t j = j0 + tid;
            const float4 f = make_float4(fx[j], fy[j], 0.f, 0.f);
            tile[tid] = FieldSrc{(double)x[j], (double)y[j], (double)f.x, (double)f.y, f};
            sfx += (double)f.x;
            sfy += (double)f.y;
        }
        __syncthreads();
        bool far = false;
        for (int k = 0; k < m; ++k) {
            const FieldSrc s = tile[k];
#pragma unroll
            for (int q = 0; q < TPL; ++q) {
                const double dxd = X[q] - s.x, dyd = Y[q] - s.y;
                const float dx = (float)dxd * rho, dy = (float)dyd * rho;
                const uint32_t bits = __builtin_bit_cast(uint32_t, fmaf(dx, dx, fmaf(dy, dy, 1.0f)));
                const uint32_t id = bits >> TAB_SHIFT;
                far = far || id >= TAB_END;
                const FieldE& e = tb[min(id, TAB_END) - TAB_BIAS];
                const float uu = tab_u(bits);
                const float4 h = e.h, g = e.g, w = e.w;
                const float Ht = fmaf(fmaf(fmaf(h.w, uu, h.z), uu, h.y), uu, h.x);
                const float H2 = fmaf(fmaf(fmaf(g.w, uu, g.z), uu, g.y), uu, g.x);
                const float wt = fmaf(fmaf(fmaf(w.w, uu, w.z), uu, w.y), uu, w.x);
                const float h2fd = H2 * fmaf(s.f.x, dx, s.f.y * dy);
                su[q] += (double)fmaf(Ht, s.f.x, h2fd * dx);
                sv[q] += (double)fmaf(Ht, s.f.y, h2fd * dy);
                sp[q] = fma(fma(s.fx, dxd, s.fy * dyd), (double)wt, sp[q]);
            }
        }
        if (__any(far)) {
            // pairs beyond the tables (or not finite), evaluated directly
            for (int k = 0; k < m; ++k) {
                const FieldSrc s = tile[k];
#pragma unroll
                for (int q = 0; q < TPL; ++q) {
                    const double dxd = X[q] - s.x, dyd = Y[q] - s.y;
                    const float dx = (float)dxd, dy = (float)dyd, sx = dx * rho, sy = dy * rho;
                    const uint32_t bits = __builtin_bit_cast(uint32_t, fmaf(sx, sx, fmaf(sy, sy, 1.0f)));
                    if ((bits >> TAB_SHIFT) < TAB_END) continue;
                    const FieldFar f = field_far(fc, fmaf(dx, dx, dy * dy), fma(dxd, dxd, dyd * dyd));
                    const float h2fd = f.H2 * fmaf(s.f.x, dx, s.f.y * dy);
                    su[q] += (double)fmaf(f.Ht, s.f.x, h2fd * dx);
                    sv[q] += (double)fmaf(f.Ht, s.f.y, h2fd * dy);
                    sp[q] = fma(fma(s.fx, dxd, s.fy * dyd), f.w, sp[q]);
                }
            }
        }
    }
    // the forces' sum, for the constant part H1(0)
    sfx = wave_total(sfx);
    sfy = wave_total(sfy);
    __syncthreads();
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = sfx;
        red[1][tid >> 6] = sfy;
    }
    __syncthreads();
    sfx = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    sfy = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    static_assert(FIELD_TILE == 256, "four waves");
#pragma unroll
    for (int q = 0; q < TPL; ++q) {
        if (a[q] < nt) {
            u[a[q]] = (float)fma(fc.h1c, sfx, su[q]);
            v[a[q]] = (float)fma(fc.h1c, sfy, sv[q]);
            p[a[q]] = (float)sp[q];
        }
    }
}

// FP64 fields: the kernel from the system's FP64 table (direct beyond it), or
// DIRECT evaluated throughout; the pressure weight directly
template <bool DIRECT>
__global__ __launch_bounds__(FIELD_TILE) void k_flow_field64(int64_t n, const double* x, const double* y,
                                                             const double* fx, const double* fy, FieldConst fc,
                                                             int64_t nt, const double* tx, const double* ty, double* u,
                                                             double* v, double* p, const TabSys64* tab)
{
    __shared__ Src4<double> tile[FIELD_TILE];
    const int tid = threadIdx.x;
    const int64_t a = (int64_t)blockIdx.x * FIELD_TILE + tid;
    const bool live = a < nt;
    const double X = live ? tx[a] : 0.0, Y = live ? ty[a] : 0.0;
    double su = 0.0, sv = 0.0, sp = 0.0, sfx = 0.0, sfy = 0.0;
    for (int64_t j0 = 0; j0 < n; j0 += FIELD_TILE) {
        const int m = (int)min<int64_t>(FIELD_TILE, n - j0);
        __syncthreads();
        if (tid < m) tile[tid] = Src4<double>{x[j0 + tid], y[j0 + tid], fx[j0 + tid], fy[j0 + tid]};
        __syncthreads();
        for (int k = 0; k < m; ++k) {
            const Src4<double> s = tile[k];
            sfx += s.fx;
            sfy += s.fy;
            const double dx = X - s.x, dy = Y - s.y, t = fma(dx, dx, dy * dy), fd = fma(s.fx, dx, s.fy * dy);
            double Ht, H2;
            if constexpr (DIRECT) {
                kernel_eval_closed<double>(fc.c64, t, Ht, H2);
            } else if (tab64_lookup(tab, t, fc.c64.ts, Ht, H2)) {
                const V2<double> d = kernel_far64(fc.c64, t);
                Ht = d.x;
                H2 = d.y;
            }
            su += fma(Ht, s.fx, H2 * fd * dx);
            sv += fma(Ht, s.fy, H2 * fd * dy);
            sp = fma(s.fx * dx + s.fy * dy, field_weight(fc, t), sp);
        }
    }
    if (live) {
        u[a] = fma(fc.h1c, sfx, su);
        v[a] = fma(fc.h1c, sfy, sv);
        p[a] = sp;
    }
}

}  // namespace

// A table costs an upload, the constants' launch and 704 intervals' set-up, 25 us.
// The Stokes limits' closed forms are a logarithm and a few products, less than
// a pair's nine table reads (512 sources, 3e5 targets: 1.34 ms direct, 2.17 from
// the table); the reading's Bessel functions are more (5.97 ms, 3.56 from the
// table), but not for few sources, whose chain of pairs is short (64 sources, 100
// targets 156 us against 126; one source and target 13 against 37).  The paper's
// blob at alpha > 0 has no closed form.  The number of targets has no say, so that
// a target's bits do not depend on the others.
bool field_direct64(const FieldConst& fc, int64_t n)
{
    return fc.c64.paper != 2.0 && (fc.stokes || n < 32);
}

hipError_t launch_flow_field(int dtype, int64_t n, const void* x, const void* y, const void* fx, const void* fy,
                             const FieldConst& fc, const FieldConst* fc_dev, int64_t nt, const void* tx, const void* ty,
                             void* u, void* v, void* p, const void* tab, void* wtab, hipStream_t st)
{
    if (nt == 0) return hipSuccess;
    if (dtype == 0) {
        hipLaunchKernelGGL(k_weight_table, dim3(TAB_N / 256 + 1), dim3(256), 0, st, fc_dev, (float4*)wtab);
        const float *X = (const float*)x, *Y = (const float*)y, *FX = (const float*)fx, *FY = (const float*)fy;
        // two targets per thread from 2^18 targets on (four workgroups per CU)
        if (nt >= (1 << 18))
            hipLaunchKernelGGL(k_flow_field32<2>, dim3((unsigned)((nt + 2 * FIELD_TILE - 1) / (2 * FIELD_TILE))),
                               dim3(FIELD_TILE), 0, st, n, X, Y, FX, FY, fc_dev, nt, (const float*)tx, (const float*)ty,
                               (float*)u, (float*)v, (float*)p, (const TabSys*)tab, (const float4*)wtab);
        else
            hipLaunchKernelGGL(k_flow_field32<1>, dim3((unsigned)((nt + FIELD_TILE - 1) / FIELD_TILE)),
                               dim3(FIELD_TILE), 0, st, n, X, Y, FX, FY, fc_dev, nt, (const float*)tx, (const float*)ty,
                               (float*)u, (float*)v, (float*)p, (const TabSys*)tab, (const float4*)wtab);
    } else {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)((nt + FIELD_TILE - 1) / FIELD_TILE)), dim3(FIELD_TILE), 0, st, n,
                               (const double*)x, (const double*)y, (const double*)fx, (const double*)fy, fc, nt,
                               (const double*)tx, (const double*)ty, (double*)u, (double*)v, (double*)p,
                               (const TabSys64*)tab);
        };
        if (tab)
            launch(k_flow_field64<false>);
        else
            launch(k_flow_field64<true>);
    }
    return hipGetLastError();
}

}  // namespace swim
