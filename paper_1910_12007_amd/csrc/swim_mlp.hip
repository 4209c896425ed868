// swim_mlp.hip -- gfx950 kernels of the MLP surrogate: fused inference (all
// layers per workgroup), a training step in two launches (the whole network
// forward and back per block of rows; weight gradients with Adam), and the
// data preparation, prescreen distance and compaction around them.
//
// Every GEMM operand is rounded to bfloat16 (nearest, ties to even) and
// products accumulate in FP32 on MFMA; FP32 master weights are kept for Adam.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include "swim_internal.h"
#include "swim_philox.h"

namespace swim {

typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// erf by Abramowitz & Stegun, Handbook of Mathematical Functions, 7.1.26:
// erf(x) = 1 - (a1 t + a2 t^2 + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x),
// x >= 0, odd extension; absolute error at most 1.5e-7 (plus the hardware
// reciprocal and exp2 at 1 ulp each), far below the BF16 resolution at which
// every activation feeds the next layer.  About 12 instructions against ~44
// for the library erff, which bound the fused MLP on the vector ALUs.
__device__ __forceinline__ float erf_as(float x)
{
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
    float p = fmaf(1.061405429f, t, -1.453152027f);
    p = fmaf(p, t, 1.421413741f);
    p = fmaf(p, t, -0.284496736f);
    p = fmaf(p, t, 0.254829592f);
    p *= t;
    const float e = __builtin_amdgcn_exp2f(-ax * ax * 1.4426950408889634f);  // exp(-x^2)
    return copysignf(fmaf(-p, e, 1.0f), x);
}

// GELU(x) = (x/2)(1 + erf(x/sqrt 2)) with erf from 7.1.26 rearranged: with
// a = |x|, z = a/sqrt 2 and erf(z) = 1 - P(t) exp(-z^2), t = 1/(1 + p z),
// GELU(x) = max(x, 0) - (a/2) P(t) exp(-a^2/2) for either sign of x (no
// copysign, no 1 + erf); the same function as (x/2)(1 + erf_as(x/sqrt 2)).
__device__ __forceinline__ float gelu_f(float x)
{
    const float a = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, a, 1.0f));
    float p = fmaf(1.061405429f, t, -1.453152027f);
    p = fmaf(p, t, 1.421413741f);
    p = fmaf(p, t, -0.284496736f);
    p = fmaf(p, t, 0.254829592f);
    // exp(-a^2/2) / 2, the halving folded into the exponent
    const float e = __builtin_amdgcn_exp2f(fmaf(a * a, -0.5f * 1.4426950408889634f, -1.0f));
    // max(x, 0) on the bits: fmaxf takes another operation to quiet its operand
    // (a NaN comes through the product either way)
    const float r = __builtin_bit_cast(float, max(__builtin_bit_cast(int, x), 0));
    return fmaf(-(a * t), p * e, r);
}

__device__ __forceinline__ float gelu_grad_f(float x)
{
    const float cdf = 0.5f * (1.0f + erf_as(x * 0.70710678118654752f));
    const float pdf = 0.39894228040143268f * __builtin_amdgcn_exp2f(-0.5f * x * x * 1.4426950408889634f);
    return fmaf(x, pdf, cdf);
}

__device__ __forceinline__ float mlp_wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Stream compaction of keep[0..n) into idx (ascending): counts per block of
// 16 waves, each wave a contiguous span of `per` flags, then the scatter,
// whose blocks add the counts before theirs (at most 1024 of them: `per`
// grows with n).  Bound by two launches: 1M flags take 2 x 5 us; with a
// serial scan of the block counts between them, one thread, 417 us.
constexpr int CMP_WAVES = 16, CMP_BLOCKS = 1024;

// flags set in this wave's span [i0, i0 + per) (uniform over the wave)
__device__ __forceinline__ int cmp_count(int64_t n, const uint8_t* keep, int64_t i0, int per, int lane)
{
    int c = 0;
    for (int k = 0; k < per; k += 64) {
        const int64_t i = i0 + k + lane;
        c += __popcll(__ballot(i < n && keep[i]));
    }
    return c;
}

__global__ __launch_bounds__(64 * CMP_WAVES) void k_count_blocks(int64_t n, const uint8_t* keep, int per,
                                                                 int32_t* counts)
{
    __shared__ int32_t s[CMP_WAVES];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c = cmp_count(n, keep, ((int64_t)blockIdx.x * CMP_WAVES + w) * per, per, lane);
    if (lane == 0) s[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int k = 0; k < CMP_WAVES; ++k) t += s[k];
        counts[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(64 * CMP_WAVES) void k_scatter(int64_t n, const uint8_t* keep, int per,
                                                            const int32_t* counts, int64_t* idx, int64_t* total)
{
    __shared__ int32_t s[CMP_WAVES];
    __shared__ int64_t before[CMP_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t i0 = ((int64_t)blockIdx.x * CMP_WAVES + w) * per;
    const int own = cmp_count(n, keep, i0, per, lane);
    int64_t c = tid < (int)blockIdx.x ? counts[tid] : 0;  // blocks before this one
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
    if (lane == 0) {
        s[w] = own;
        before[w] = c;
    }
    __syncthreads();
    int64_t at = 0, end = 0;
    for (int k = 0; k < CMP_WAVES; ++k) {
        at += before[k] + (k < w ? s[k] : 0);
        end += before[k] + s[k];
    }
    for (int k = 0; k < per; k += 64) {
        const int64_t i = i0 + k + lane;
        const uint64_t m = __ballot(i < n && keep[i]);
        if ((m >> lane) & 1) idx[at + __popcll(m & ((1ull << lane) - 1))] = i;
        at += __popcll(m);
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) *total = end;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_compact(int64_t n, const uint8_t* keep, int32_t* counts, int64_t* idx, int64_t* total, hipStream_t st)
{
    const int64_t per = 64 * std::max<int64_t>(4, (n + 64 * CMP_WAVES * CMP_BLOCKS - 1) / (64 * CMP_WAVES * CMP_BLOCKS));
    const unsigned nb = (unsigned)((n + CMP_WAVES * per - 1) / (CMP_WAVES * per));
    hipLaunchKernelGGL(k_count_blocks, dim3(nb), dim3(64 * CMP_WAVES), 0, st, n, keep, (int)per, counts);
    hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(64 * CMP_WAVES), 0, st, n, keep, (int)per, counts, idx, total);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// surrogate data preparation
// ---------------------------------------------------------------------------
// X[i] = (alpha, ln S_b, ln S_s, b, omega), standardized when mu/sd are given
__global__ void k_features(int64_t n, const double* theta, double b, double om, const float* mu, const float* sd,
                           float* X)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double f[5] = {theta[3 * i], log(theta[3 * i + 1]), log(theta[3 * i + 2]), b, om};
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        float v = (float)f[c];
        if (mu) v = (v - mu[c]) / sd[c];
        X[i * 5 + c] = v;
    }
}

// T[i] = (head displacement at the chosen samples, x then y, ..., speed)
template <typename T>
__global__ void k_targets(int64_t n, int n_obs, const T* obs, const T* speed, double x0, double y0, const int32_t* idx,
                          int n_sum, float* Tout)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int nt = 2 * n_sum + 1;
    for (int j = 0; j < n_sum; ++j) {
        const T* o = obs + (i * n_obs + idx[j]) * 2;
        Tout[i * nt + 2 * j] = (float)((double)o[0] - x0);
        Tout[i * nt + 2 * j + 1] = (float)((double)o[1] - y0);
    }
    Tout[i * nt + 2 * n_sum] = (float)speed[i];
}

// column mean and standard deviation (population), one workgroup per column,
// fixed summation order
__global__ __launch_bounds__(256) void k_colstats(int64_t n, int cols, const float* A, float* mu, float* sd)
{
    __shared__ double red[256];
    const int c = blockIdx.x;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)A[i * cols + c];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const double m = red[0] / (double)n;
    __syncthreads();
    double q = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double d = (double)A[i * cols + c] - m;
        q += d * d;
    }
    red[threadIdx.x] = q;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        mu[c] = (float)m;
        const double v = red[0] / (double)n;
        sd[c] = v > 0.0 ? (float)sqrt(v) : 1.0f;
    }
}

__global__ void k_standardize(int64_t n, int cols, float* A, const float* mu, const float* sd)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * cols) return;
    const int c = (int)(e % cols);
    A[e] = (A[e] - mu[c]) / sd[c];
}

// prior draws on the device, identical to the host abc_prior_draw:
// theta[i][d] = lo[d] + (hi[d] - lo[d]) u_d, u from Philox stream 0, draws 0, 1
__global__ void k_prior_draw(uint64_t seed, int64_t n, double lo0, double lo1, double lo2, double hi0, double hi1,
                             double hi2, double* theta)
{
    // separately rounded multiply and add, as the host draw computes them
    // (the default contraction would fuse them into one FMA)
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double u[4];
    philox_uniforms2(seed, 0, (uint64_t)i, 0, u);
    philox_uniforms2(seed, 0, (uint64_t)i, 1, u + 2);
    const double lo[3] = {lo0, lo1, lo2}, hi[3] = {hi0, hi1, hi2};
#pragma unroll
    for (int d = 0; d < 3; ++d) theta[3 * i + d] = lo[d] + (hi[d] - lo[d]) * u[d];
}

// param rows (alpha, S_b, S_s, b, omega, k, 0, 0, 0) of the theta rows idx[j]
// (idx NULL: j itself), j < *n_dev; an index outside [0, n_theta) gives a
// NaN row (that system is then flagged SWIM_ST_BADPARAM)
__global__ void k_param_rows(int64_t cap, const int64_t* n_dev, const int64_t* idx, int64_t n_theta,
                             const double* theta, double b, double om, double kw, double* rows)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= cap || (n_dev && j >= *n_dev)) return;
    const int64_t i = idx ? idx[j] : j;
    const bool ok = i >= 0 && i < n_theta;
    double* P = rows + 9 * j;
    P[0] = ok ? theta[3 * i] : NAN;
    P[1] = ok ? theta[3 * i + 1] : NAN;
    P[2] = ok ? theta[3 * i + 2] : NAN;
    P[3] = b;
    P[4] = om;
    P[5] = kw;
    P[6] = 0.0;
    P[7] = 0.0;
    P[8] = 0.0;
}

// dst[j] = src[idx[j]] (rows of `cols` floats), j < *n_dev; an index outside
// [0, n_src) gives a NaN row
__global__ void k_gather_f32(int64_t cap, const int64_t* n_dev, const int64_t* idx, int64_t n_src, const float* src,
                             int cols, float* dst)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t j = e / cols;
    if (j >= cap || j >= *n_dev) return;
    const int c = (int)(e % cols);
    const int64_t i = idx[j];
    dst[j * cols + c] = (i >= 0 && i < n_src) ? src[i * cols + c] : NAN;
}

__global__ void k_flag_eq(int64_t n, const int32_t* v, int32_t want, uint8_t* keep)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) keep[i] = v[i] == want ? 1 : 0;
}

// keep[i] &= every one of the first n_disp entries of row i of T is finite
// with magnitude <= max_disp
__global__ void k_flag_bounded(int64_t n, const float* T, int nt, int n_disp, float max_disp, uint8_t* keep)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    bool ok = keep[i] != 0;
    for (int j = 0; j < n_disp; ++j) ok = ok && fabsf(T[i * nt + j]) <= max_disp;
    keep[i] = ok ? 1 : 0;
}

hipError_t launch_features(int64_t n, const double* theta, double b, double om, const float* mu, const float* sd,
                           float* X, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, theta, b, om, mu, sd, X);
    return hipGetLastError();
}

hipError_t launch_targets(int dtype, int64_t n, int n_obs, const void* obs, const void* speed, double x0, double y0,
                          const int32_t* idx, int n_sum, float* T, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const dim3 g((unsigned)((n + 255) / 256));
    if (dtype == 0)
        hipLaunchKernelGGL(k_targets<float>, g, dim3(256), 0, st, n, n_obs, (const float*)obs, (const float*)speed, x0,
                           y0, idx, n_sum, T);
    else
        hipLaunchKernelGGL(k_targets<double>, g, dim3(256), 0, st, n, n_obs, (const double*)obs, (const double*)speed,
                           x0, y0, idx, n_sum, T);
    return hipGetLastError();
}

hipError_t launch_colstats(int64_t n, int cols, const float* A, float* mu, float* sd, hipStream_t st)
{
    hipLaunchKernelGGL(k_colstats, dim3(cols), dim3(256), 0, st, n, cols, A, mu, sd);
    return hipGetLastError();
}

hipError_t launch_standardize(int64_t n, int cols, float* A, const float* mu, const float* sd, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_standardize, dim3((unsigned)((n * cols + 255) / 256)), dim3(256), 0, st, n, cols, A, mu, sd);
    return hipGetLastError();
}

hipError_t launch_prior_draw(uint64_t seed, int64_t n, const double* lo, const double* hi, double* theta,
                             hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prior_draw, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, seed, n, lo[0], lo[1], lo[2],
                       hi[0], hi[1], hi[2], theta);
    return hipGetLastError();
}

hipError_t launch_param_rows(int64_t cap, const int64_t* n_dev, const int64_t* idx, int64_t n_theta,
                             const double* theta, double b, double om, double kw, double* rows, hipStream_t st)
{
    if (cap <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_param_rows, dim3((unsigned)((cap + 255) / 256)), dim3(256), 0, st, cap, n_dev, idx, n_theta,
                       theta, b, om, kw, rows);
    return hipGetLastError();
}

hipError_t launch_gather_f32(int64_t cap, const int64_t* n_dev, const int64_t* idx, int64_t n_src, const float* src,
                             int cols, float* dst, hipStream_t st)
{
    if (cap <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_f32, dim3((unsigned)((cap * cols + 255) / 256)), dim3(256), 0, st, cap, n_dev, idx,
                       n_src, src, cols, dst);
    return hipGetLastError();
}

hipError_t launch_flag_eq(int64_t n, const int32_t* v, int32_t want, uint8_t* keep, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_flag_eq, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, v, want, keep);
    return hipGetLastError();
}

hipError_t launch_flag_bounded(int64_t n, const float* T, int nt, int n_disp, float max_disp, uint8_t* keep,
                               hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_flag_bounded, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, T, nt, n_disp,
                       max_disp, keep);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fused inference: every workgroup carries MLP_RT = 64 rows through all
// five layers, one 16-row tile per wave, with the activations in
// registers.  The product is formed transposed, C^T = W^T H^T, with
// v_mfma_f32_16x16x32_bf16: the weights are the A operand (rows n), the
// activations the B operand (columns = rows m of the batch).  A lane's four
// results of output tile c are the outputs n = 16c + 4q + r (q = lane / 16,
// r = 0..3) of row m = lane % 16; bias, GELU and the rounding to bfloat16
// turn tiles 2p and 2p + 1 into the lane's eight operand values of the next
// layer's k slice p, i.e. the k order within each 32-wide slice is
//   slot 8q + j  <->  k = 4q + j (j < 4),  16 + 4q + (j - 4) (j >= 4),
// and the packed weights (k_pack_w16) use the same order.  So activations
// never touch LDS; the weights, a bfloat16 copy packed as operand fragments (k
// padded to a multiple of 32, n of the last layer to 48), pass through LDS in
// chunks of MLP_KC = 32 k, double-buffered: the next chunk (of this layer or
// the next) goes from L2 to LDS by loads that take no registers while the
// current one feeds the MFMAs, and a fragment is read in lane order, without
// bank conflicts or address arithmetic.  FP32 accumulation over the slices in
// order.  MODE 0 writes the outputs; MODE 1 computes the prescreen distance of
// every row.
// Bound by the vector ALUs: 14 operations per activation, two of them at a
// quarter of the rate, are 0.55 ms for 1M rows; the MFMAs' 0.18 and the weights'
// way out of LDS, 0.35, hide behind them only in other waves, so the count of
// waves decides: 126 VGPRs and 32 KB, four per SIMD.  One prescreen of 1M rows
// takes 700..754 us by the box (714 on the one of the next figures); with the chunks through registers and padded rows (166 VGPRs,
// three waves) 981; with 64-bit addresses per lane for the loads 756 at three
// waves, 855 at four, with spills.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
constexpr int MLP_RT = 64, MLP_KC = 32;
constexpr int MLP_NL = 5;
constexpr int mlp_kp(int l) { return l == 0 ? 32 : 256; }   // padded K
constexpr int mlp_np(int l) { return l == MLP_NL - 1 ? 48 : 256; }  // padded N
constexpr int mlp_k(int l) { return l == 0 ? 5 : 256; }
constexpr int mlp_n(int l) { return l == MLP_NL - 1 ? 33 : 256; }
constexpr int64_t mlp_w16_off(int l)
{
    int64_t o = 0;
    for (int k = 0; k < l; ++k) o += (int64_t)mlp_np(k) * mlp_kp(k);
    return o;
}
constexpr int64_t MLP_W16_TOTAL = mlp_w16_off(MLP_NL);
constexpr int64_t mlp_offW_d(int l)
{
    int64_t o = 0;
    for (int k = 0; k < l; ++k) o += (int64_t)mlp_k(k) * mlp_n(k) + mlp_n(k);
    return o;
}
// the k of operand slot s (0..31) of a 32-wide slice (see above)
__host__ __device__ constexpr int mlp_slot_k(int s)
{
    return (s & 7) < 4 ? 4 * (s >> 3) + (s & 7) : 16 + 4 * (s >> 3) + (s & 7) - 4;
}

// bfloat16 copy of the weights, transposed, k in slot order, padded (zeros),
// as operand fragments: chunk by chunk, tile by tile, the eight values of each
// lane in a row
__global__ void k_pack_w16(const float* P, uint16_t* W16)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= MLP_W16_TOTAL) return;
    int l = 0;
    while (l + 1 < MLP_NL && e >= mlp_w16_off(l + 1)) ++l;
    const int i = (int)(e - mlp_w16_off(l)), nt = mlp_np(l) / 16;
    const int j = i & 7, lane = (i >> 3) & 63, tile = (i >> 9) % nt, chunk = (i >> 9) / nt;
    const int n = 16 * tile + (lane & 15), k = MLP_KC * chunk + mlp_slot_k(8 * (lane >> 4) + j);
    const float v = (n < mlp_n(l) && k < mlp_k(l)) ? P[mlp_offW_d(l) + (int64_t)k * mlp_n(l) + n] : 0.0f;
    W16[e] = f2bf(v);
}

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// one chunk of NP fragments (1 KB each) at byte `at` of the packed weights,
// from L2 into LDS without registers; complete behind this wave's wait and the
// workgroup's barrier (chunk_ready)
#if defined(__HIP_DEVICE_COMPILE__)
typedef __amdgpu_buffer_rsrc_t WBuf;
__device__ __forceinline__ WBuf wbuf(const uint16_t* W16)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(W16), 0, (int)(MLP_W16_TOTAL * 2), 0x00020000);
}
#else
typedef const uint16_t* WBuf;
__device__ inline WBuf wbuf(const uint16_t* W16) { return W16; }
#endif
template <int NP> __device__ __forceinline__ void chunk_fetch(WBuf W, int at, uint16_t* to, int wave, int lane)
{
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int i = 0; i < (NP + 3) / 4; ++i) {
        const int piece = wave + 4 * i;
        if (NP % 4 == 0 || piece < NP)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(W, (__attribute__((address_space(3))) void*)(to + 512 * piece), 16,
                                                     16 * lane, at + 1024 * piece, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);  // not behind the products that hide it
#endif
}
__device__ __forceinline__ void chunk_ready()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
    __syncthreads();
}
__device__ __forceinline__ uint32_t pack_bf2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, bf16x2_t{(__bf16)a, (__bf16)b});
}
// acc[c] += chunk's tile c times the row tile's slice h
template <int NT>
__device__ __forceinline__ void chunk_mfma(const uint16_t* Ws, u32x4_t h, int lane, f32x4_t (&acc)[16])
{
    const bf16x8_t hv = __builtin_bit_cast(bf16x8_t, h);
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        const bf16x8_t wv = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(Ws + 512 * c + 8 * lane));
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, hv, acc[c], 0, 0, 0);
    }
}
// GELU, bfloat16: tiles 2p, 2p + 1 -> slice p of the next layer's operand
__device__ __forceinline__ void mlp_activate(const f32x4_t (&acc)[16], u32x4_t (&h)[8])
{
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const f32x4_t a0 = acc[2 * p], a1 = acc[2 * p + 1];
        h[p] = u32x4_t{pack_bf2(gelu_f(a0[0]), gelu_f(a0[1])), pack_bf2(gelu_f(a0[2]), gelu_f(a0[3])),
                       pack_bf2(gelu_f(a1[0]), gelu_f(a1[1])), pack_bf2(gelu_f(a1[2]), gelu_f(a1[3]))};
    }
}

template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_mlp_fused(
    int64_t M, const float* __restrict__ X, const uint16_t* __restrict__ W16, const float* __restrict__ P,
    float* __restrict__ Y, const float* __restrict__ out_mu, const float* __restrict__ out_sd,
    const float* __restrict__ obs, int n_sum, float tol, float* __restrict__ dist, uint8_t* __restrict__ keep)
{
    __shared__ __align__(16) uint16_t Wa[16 * 512], Wb[16 * 512];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;
    // this lane's row of the batch
    const int64_t row = (int64_t)blockIdx.x * MLP_RT + 16 * wave + (lane & 15);
    const WBuf W = wbuf(W16);
    int next = 0;  // byte of the chunk fetched next
    chunk_fetch<16>(W, next, Wa, wave, lane);
    next += 16 * 1024;
    f32x4_t acc[16];
    u32x4_t h[8];
    // hidden layers start from the bias (C^T[n][m] = b[n])
    auto from_bias = [&](int l) {
        const float* bias = P + mlp_offW_d(l) + (int64_t)mlp_k(l) * mlp_n(l);
#pragma unroll
        for (int c = 0; c < 16; ++c) acc[c] = *reinterpret_cast<const f32x4_t*>(bias + 16 * c + 4 * q);
    };
    {
        // layer 0: the five inputs in slot order, zeros elsewhere
        float xin[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = mlp_slot_k(8 * q + j);
            xin[j] = (k < 5 && row < M) ? X[row * 5 + k] : 0.0f;
        }
        from_bias(0);
        chunk_ready();
        chunk_fetch<16>(W, next, Wb, wave, lane);
        next += 16 * 1024;
        chunk_mfma<16>(Wa, u32x4_t{pack_bf2(xin[0], xin[1]), pack_bf2(xin[2], xin[3]), pack_bf2(xin[4], xin[5]),
                                   pack_bf2(xin[6], xin[7])},
                       lane, acc);
        mlp_activate(acc, h);
    }
    // chunk c of layers 1.. lies in Wb (c even) or Wa (c odd)
#pragma unroll 1
    for (int l = 1; l < MLP_NL - 1; ++l) {
        from_bias(l);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            chunk_ready();  // chunk c there; nobody reads the other buffer any more
            if (c < 7 || l + 1 < MLP_NL - 1)
                chunk_fetch<16>(W, next, c & 1 ? Wb : Wa, wave, lane);
            else
                chunk_fetch<3>(W, next, Wb, wave, lane);
            next += 16 * 1024;
            chunk_mfma<16>(c & 1 ? Wa : Wb, h[c], lane, acc);
        }
        mlp_activate(acc, h);
    }
    next = (int)(mlp_w16_off(MLP_NL - 1) * 2) + 3 * 1024;
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        chunk_ready();
        if (c < 7) chunk_fetch<3>(W, next + 3 * 1024 * c, c & 1 ? Wb : Wa, wave, lane);
        chunk_mfma<3>(c & 1 ? Wa : Wb, h[c], lane, acc);
    }
    const float* bias = P + mlp_offW_d(MLP_NL - 1) + (int64_t)mlp_k(MLP_NL - 1) * mlp_n(MLP_NL - 1);
    if constexpr (MODE == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = 16 * c + 4 * q + r;
                if (n < 33 && row < M) Y[row * 33 + n] = acc[c][r] + bias[n];
            }
    } else {
        // prescreen: d = sqrt(mean_{n < n_sum} (mu_n + sd_n y_n - obs_n)^2)
        float sq = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = 16 * c + 4 * q + r;
                if (n < n_sum) {
                    const float dv = fmaf(out_sd[n], acc[c][r] + bias[n], out_mu[n]) - obs[n];
                    sq = fmaf(dv, dv, sq);
                }
            }
        // the four lanes of row m (lane % 16 equal), fixed order
        sq += __shfl_xor(sq, 16, 64);
        sq += __shfl_xor(sq, 32, 64);
        if (q == 0 && row < M) {
            const float d = sqrtf(sq / (float)n_sum);
            if (dist) dist[row] = d;
            keep[row] = (d <= tol) ? 1 : 0;
        }
    }
}

// ---------------------------------------------------------------------------
// Training step in two launches.
//
// k_mlp_step carries 16 RT rows through the whole network and back, one
// workgroup of 16 waves: wave w owns features 16w..16w+15 of every hidden
// layer, with v_mfma_f32_16x16x16bf16_1k (A = rows, B = weights).  The
// activations pass between layers as bfloat16 through LDS, in the MFMA's
// operand order (8 KB per 16 rows, double-buffered); pre-activations stay in
// registers for gelu' on the way back; the weights come straight from L2 as
// bfloat16 operand fragments (one 16-byte load per lane and 32 k), the next
// layer's loaded ahead of the barrier.  It leaves bfloat16 copies of the
// activations and of the gradients dA_l, feature-major, the gradients also in
// FP32 (for the biases), and per-workgroup sums of the squared error.
//
// k_mlp_update forms the weight gradients dW_l = H_{l-1}^T dA_l: one workgroup
// of 16 waves per 32 x 32 tile, wave z summing slice z of the rows, the slices
// added in order through LDS; the same workgroup then takes the tile's Adam
// step and refreshes the packed bfloat16 weights (or, for surrogate_grad,
// writes the gradient).  Bias gradients and the loss take a few more
// workgroups of the same launch.
//
// A batch of 1024 rows is 1.3 GFLOP, under 1 us of MFMA time: a step is bound
// by launches and by the serial chain of nine layers, so there are two
// launches (29 with one GEMM, reduction, column sum, gather and Adam kernel
// each: 170 us a step) and nothing of a layer leaves the workgroup before the
// next one needs it.  Rows per workgroup: 16 fill four times as many CUs at
// the batch of 1024; from 8192 rows on, 32 halve the weights' L2 traffic.
//
// Sums over k run in slices of kper 32-wide chunks, each slice from zero, the
// slices added in order (MlpSplit): the order the FP32 accumulation has had
// with split-K launches, so a change of launch shape does not change a bit.
// ---------------------------------------------------------------------------
constexpr int MLP_HID = 256, MLP_OUTN = 33;  // hidden features, outputs
// packed weights: forward B operands of layers 0..4, then backward ones of
// layers 1..4; one fragment = 64 lanes x 8 values (layer 0: x 4)
constexpr int64_t MLP_WB0 = 0, MLP_WB1 = 16 * 64 * 4, MLP_WB4 = MLP_WB1 + 3 * 65536,
                  MLP_WT1 = MLP_WB4 + 3 * 8 * 512, MLP_WT4 = MLP_WT1 + 3 * 65536,
                  MLP_WPK = MLP_WT4 + 16 * 2 * 512;

// place of value (red, col) in a layer's fragments: red the summed index (nsp
// 32-wide pieces of it), col the output feature
__host__ __device__ constexpr int mlp_frag(int red, int col, int nsp)
{
    return (((col >> 4) * nsp + (red >> 5)) * 64 + (col & 15) + 16 * ((red >> 2) & 3)) * 8 + ((red >> 4) & 1) * 4 +
           (red & 3);
}

__global__ void k_mlp_pack(const float* __restrict__ P, uint16_t* __restrict__ W)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= MLP_WPK) return;
    float v = 0.0f;
    if (e < MLP_WB1) {
        const int j = e & 3, lane = (e >> 2) & 63, n = (int)(e >> 8) * 16 + (lane & 15), k = 4 * (lane >> 4) + j;
        if (k < 5) v = P[mlp_offW_d(0) + (int64_t)k * MLP_HID + n];
    } else {
        // region start, layer, pieces of the summed index, forward or backward
        const bool fwd = e < MLP_WT1;
        const int64_t r0 = e < MLP_WB4 ? MLP_WB1 : fwd ? MLP_WB4 : e < MLP_WT4 ? MLP_WT1 : MLP_WT4;
        const bool hid = r0 == MLP_WB1 || r0 == MLP_WT1;
        const int l = hid ? 1 + (int)((e - r0) >> 16) : 4;
        const int i = (int)(hid ? (e - r0) & 65535 : e - r0), nsp = (hid || fwd) ? 8 : 2;
        const int x = i & 7, lane = (i >> 3) & 63, t = i >> 9;
        const int red = 32 * (t % nsp) + 16 * (x >> 2) + 4 * (lane >> 4) + (x & 3), col = 16 * (t / nsp) + (lane & 15);
        const int k = fwd ? red : col, n = fwd ? col : red, N = l == 4 ? MLP_OUTN : MLP_HID;
        if (n < N) v = P[mlp_offW_d(l) + (int64_t)k * N + n];
    }
    W[e] = f2bf(v);
}

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// Features stored feature-major: row R of a batch sits at mlp_rowpos(R) of
// its feature's Mpad values, in the order a lane's 16-byte load takes it as
// the operand of two 16-row MFMAs
__device__ __forceinline__ int64_t mlp_rowpos(int64_t R)
{
    return (R & ~(int64_t)31) + 8 * ((R >> 2) & 3) + 4 * ((R >> 4) & 1) + (R & 3);
}

// sum over nsp 32-wide pieces of this lane's operand pairs (a from LDS, b in
// registers), in slices of kper pieces
template <int NSP>
__device__ __forceinline__ f32x4_t mlp_dot(const u32x4_t* a, const u32x4_t (&b)[8], int kper)
{
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f}, acc = {0.f, 0.f, 0.f, 0.f};
    int left = kper;
#pragma unroll
    for (int sp = 0; sp < NSP; ++sp) {
        const u32x4_t av = a[sp * 64];
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4_t, u32x2_t{av[0], av[1]}),
                                                        __builtin_bit_cast(bf16x4_t, u32x2_t{b[sp][0], b[sp][1]}), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(bf16x4_t, u32x2_t{av[2], av[3]}),
                                                        __builtin_bit_cast(bf16x4_t, u32x2_t{b[sp][2], b[sp][3]}), acc, 0, 0, 0);
        if (--left == 0 || sp == NSP - 1) {
            sum += acc;
            acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
            left = kper;
        }
    }
    return sum;
}

template <int RT> __global__ __launch_bounds__(1024) void k_mlp_step(MlpStep a)
{
    __shared__ __align__(16) uint16_t frag[2][RT][8 * 512];  // operand fragments of the current and next layer
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * 16 * RT;
    const int n = 16 * w + c;  // this lane's feature
    // where this lane's values go: rows 4q + r of feature n
    const int fsp = w >> 1, fel = (w & 1) * 4 + (c & 3), fln = 16 * (c >> 2) + 4 * q;
    bool live[RT][4];
    int64_t pos[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        pos[t] = mlp_rowpos(row0 + 16 * t + 4 * q);
#pragma unroll
        for (int r = 0; r < 4; ++r) live[t][r] = row0 + 16 * t + 4 * q + r < a.M;
    }
    auto load_w = [&](u32x4_t (&b)[8], int64_t off, int nsp, int tile) {
        const u32x4_t* p = reinterpret_cast<const u32x4_t*>(a.W + off) + (int64_t)tile * nsp * 64 + lane;
#pragma unroll
        for (int sp = 0; sp < 8; ++sp)
            if (sp < nsp) b[sp] = p[sp * 64];
    };
    // values of this lane (4 rows of feature n) to the fragments and, with
    // rows beyond M zeroed, to the feature-major copy
    auto put = [&](int buf, int t, const float (&v)[4], uint16_t* copy, int64_t feat) {
        uint32_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h[r] = f2bf(v[r]);
            frag[buf][t][(fsp * 64 + fln + r) * 8 + fel] = (uint16_t)h[r];
            if (!live[t][r]) h[r] = 0;
        }
        *reinterpret_cast<u32x2_t*>(copy + feat * a.Mpad + pos[t]) = u32x2_t{h[0] | h[1] << 16, h[2] | h[3] << 16};
    };
    // the gradients in FP32, for the bias gradients' sums over the rows
    auto keep32 = [&](int t, const float (&v)[4], int64_t feat) {
        *reinterpret_cast<f32x4_t*>(a.DF + feat * a.Mpad + row0 + 16 * t + 4 * q) = f32x4_t{v[0], v[1], v[2], v[3]};
    };
    float pre[4][RT][4];
    u32x4_t wc[8], wn[8];
    load_w(wc, MLP_WB1, 8, w);
    // layer 0: the operand (row c, k = 4q..4q+3) straight from X
    {
        const bf16x4_t bv = __builtin_bit_cast(
            bf16x4_t, *reinterpret_cast<const u32x2_t*>(a.W + MLP_WB0 + (int64_t)(w * 64 + lane) * 4));
        const float b0 = a.P[mlp_offW_d(0) + 5 * MLP_HID + n];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int64_t R = row0 + 16 * t + c;
            float x[4] = {0.f, 0.f, 0.f, 0.f};
            if (q < 2 && R < a.M) {
                const int64_t src = a.perm ? a.perm[R] : R;
                const bool ok = src >= 0 && src < a.nrows;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * q + j < 5) x[j] = ok ? a.X[src * 5 + 4 * q + j] : NAN;
            }
            uint32_t h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = f2bf(x[j]);
            if (w == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) a.XT[(int64_t)(4 * q + j) * a.Mpad + mlp_rowpos(R)] = (uint16_t)h[j];
            }
            const f32x4_t z = {0.f, 0.f, 0.f, 0.f};
            const f32x4_t s = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                __builtin_bit_cast(bf16x4_t, u32x2_t{h[0] | h[1] << 16, h[2] | h[3] << 16}), bv, z, 0, 0, 0);
            float g[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                pre[0][t][r] = s[r] + b0;
                g[r] = gelu_f(pre[0][t][r]);
            }
            put(0, t, g, a.HT, n);
        }
    }
    // hidden layers 1..3
#pragma unroll
    for (int l = 1; l < 4; ++l) {
        const float bl = a.P[mlp_offW_d(l) + 65536 + n];
        if (l < 3)
            load_w(wn, MLP_WB1 + (int64_t)l * 65536, 8, w);
        else if (w < 3)
            load_w(wn, MLP_WB4, 8, w);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const f32x4_t s =
                mlp_dot<8>(reinterpret_cast<const u32x4_t*>(frag[(l - 1) & 1][t]) + lane, wc, a.kf);
            float g[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                pre[l][t][r] = s[r] + bl;
                g[r] = gelu_f(pre[l][t][r]);
            }
            put(l & 1, t, g, a.HT + (int64_t)l * MLP_HID * a.Mpad, n);
        }
#pragma unroll
        for (int sp = 0; sp < 8; ++sp) wc[sp] = wn[sp];
    }
    // output layer, its squared error and gradient dY = sc (Y - T): three waves;
    // features 33..63 of dY are zero
    load_w(wn, MLP_WT4, 2, w);
    __syncthreads();
    if (w < 4) {
        float sq = 0.f;
        const bool col = n < MLP_OUTN;
        const float b4 = col ? a.P[mlp_offW_d(4) + MLP_HID * MLP_OUTN + n] : 0.f;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            float d[4] = {0.f, 0.f, 0.f, 0.f};
            if (w < 3) {
                const f32x4_t s = mlp_dot<8>(reinterpret_cast<const u32x4_t*>(frag[1][t]) + lane, wc, a.ko);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (col && live[t][r]) {
                        const int64_t R = row0 + 16 * t + 4 * q + r;
                        const int64_t src = a.perm ? a.perm[R] : R;
                        const bool ok = src >= 0 && src < a.nrows;
                        const float e = (s[r] + b4) - (ok ? a.T[src * MLP_OUTN + n] : NAN);
                        d[r] = a.sc * e;
                        sq += e * e;
                    }
                }
            }
            // the fragments' next buffer is free: layer 3 read buffer 0
            if (w < 3) {
                put(0, t, d, a.YT, n);
                if (col) keep32(t, d, 4 * MLP_HID + n);
            } else
#pragma unroll
                for (int r = 0; r < 4; ++r) frag[0][t][(fsp * 64 + fln + r) * 8 + fel] = 0;
        }
        if (w < 3) {
            sq = mlp_wave_sum(sq);
            if (lane == 0) a.lossp[(int64_t)blockIdx.x * 3 + w] = sq;
        }
    }
    // back: dA_{l-1} = (dA_l W_l^T) gelu'(pre_{l-1})
#pragma unroll
    for (int l = 4; l >= 1; --l) {
#pragma unroll
        for (int sp = 0; sp < 8; ++sp) wc[sp] = wn[sp];
        if (l > 1) load_w(wn, MLP_WT1 + (int64_t)(l - 2) * 65536, 8, w);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const u32x4_t* f = reinterpret_cast<const u32x4_t*>(frag[l & 1][t]) + lane;
            const f32x4_t s = l == 4 ? mlp_dot<2>(f, wc, a.kb4) : mlp_dot<8>(f, wc, a.kb);
            float g[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                g[r] = live[t][r] ? s[r] * gelu_grad_f(pre[l - 1][t][r]) : 0.f;
            }
            put((l & 1) ^ 1, t, g, a.DT + (int64_t)(l - 1) * MLP_HID * a.Mpad, n);
            keep32(t, g, (l - 1) * MLP_HID + n);
        }
    }
}

// tiles of k_mlp_update: layers 1..3 (64 each), layer 4 (8 x 2), layer 0
// (8), then 8 bias columns a workgroup, then the loss
constexpr int MLP_UT = 3 * 64 + 16 + 8, MLP_UB = (MLP_DBN + 7) / 8;

// Adam with bias-corrected moments: p -= lr mhat / (sqrt(vhat) + eps)
__device__ __forceinline__ float mlp_adam(const MlpUpdate& u, int64_t i, float g)
{
    const float mi = fmaf(u.b1, u.m[i], (1.0f - u.b1) * g);
    const float vi = fmaf(u.b2, u.v[i], (1.0f - u.b2) * g * g);
    u.m[i] = mi;
    u.v[i] = vi;
    const float mh = mi / u.c1, vh = vi / u.c2;
    const float p = u.p[i] - u.lr * mh / (sqrtf(vh) + u.eps);
    u.p[i] = p;
    return p;
}

template <bool ADAM> __global__ __launch_bounds__(1024) void k_mlp_update(MlpUpdate u)
{
    // the waves' tiles; rotating a row's columns by 8 per four rows spreads the
    // MFMA result's rows over the banks
    __shared__ float part[16][32][32];
    auto at = [](int row, int col) { return (col + 8 * (row >> 2)) & 31; };
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int z = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = blockIdx.x;
    if (b >= MLP_UT) {
        b -= MLP_UT;
        if (b < MLP_UB) {
            // bias gradients, 8 columns a workgroup: 128 groups of rows each
            // summing every 128th row, then a fixed tree over the groups
            float(*red)[129] = reinterpret_cast<float(*)[129]>(&part[0][0][0]);
            const int g = tid & 127, n = 8 * b + (tid >> 7);
            float s = 0.f;
            if (n < MLP_DBN)
                for (int64_t m = g; m < u.M; m += 128) s += u.DF[(int64_t)n * u.Mpad + m];
            red[tid >> 7][g] = s;
            __syncthreads();
            for (int w = 64; w >= 1; w >>= 1) {
                if (g < w) red[tid >> 7][g] += red[tid >> 7][g + w];
                __syncthreads();
            }
            if (g == 0 && n < MLP_DBN) {
                const int l = n / MLP_HID;  // layers 0..3, then the 33 of layer 4
                const int64_t i = mlp_offW_d(l) + (int64_t)mlp_k(l) * mlp_n(l) + (n - l * MLP_HID);
                if (ADAM)
                    mlp_adam(u, i, red[tid >> 7][0]);
                else
                    u.g[i] = red[tid >> 7][0];
            }
        } else if (u.loss) {
            const int col = tid & 31, seg = tid >> 5;
            float s = 0.f;
            for (int64_t i = tid; i < 3 * u.nwg; i += 1024) s += u.lossp[i];
            part[0][seg][col] = s;
            __syncthreads();
            if (seg == 0) {
                s = 0.f;
                for (int k = 0; k < 32; ++k) s += part[0][k][col];
                part[1][0][col] = s;
            }
            __syncthreads();
            if (tid == 0) {
                s = 0.f;
                for (int k = 0; k < 32; ++k) s += part[1][0][k];
                *u.loss = s;
            }
        }
        return;
    }
    int l, tk, tn;
    if (b < 192) {
        l = 1 + (b >> 6);
        tk = (b >> 3) & 7;
        tn = b & 7;
    } else if (b < 208) {
        l = 4;
        tk = (b - 192) >> 1;
        tn = b & 1;
    } else {
        l = 0;
        tk = 0;
        tn = b - 208;
    }
    const int K = l == 0 ? 5 : MLP_HID, N = l == 4 ? MLP_OUTN : MLP_HID;
    const uint16_t* A = l == 0 ? u.XT : u.HT + (int64_t)(l - 1) * MLP_HID * u.Mpad;
    const uint16_t* D = l == 4 ? u.YT : u.DT + (int64_t)l * MLP_HID * u.Mpad;
    const int kper = l == 0 ? u.kw0 : l == 4 ? u.kw4 : u.kw;
    const int chunks = (int)(u.Mpad >> 5), S = (chunks + kper - 1) / kper;  // slices: at most 16
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    const u32x4_t *pa[2], *pd[2];
    bool la[2], ld[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int k = 32 * tk + 16 * t + c, n = 32 * tn + 16 * t + c;
        la[t] = k < K;
        ld[t] = n < N;
        pa[t] = reinterpret_cast<const u32x4_t*>(A + (int64_t)(la[t] ? k : 0) * u.Mpad) + q;
        pd[t] = reinterpret_cast<const u32x4_t*>(D + (int64_t)(ld[t] ? n : 0) * u.Mpad) + q;
    }
    f32x4_t acc[2][2] = {};
    if (z < S) {
        const int c1 = min(chunks, (z + 1) * kper);
        for (int ch = z * kper; ch < c1; ++ch) {
            u32x4_t av[2], dv[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                av[t] = la[t] ? pa[t][4 * ch] : zero;
                dv[t] = ld[t] ? pd[t][4 * ch] : zero;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                            __builtin_bit_cast(bf16x4_t, u32x2_t{av[i][2 * h], av[i][2 * h + 1]}),
                            __builtin_bit_cast(bf16x4_t, u32x2_t{dv[j][2 * h], dv[j][2 * h + 1]}), acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * i + 4 * q + r;
                    part[z][row][at(row, 16 * j + c)] = acc[i][j][r];
                }
    }
    __syncthreads();
    const int kk = tid >> 5, nn = tid & 31, k = 32 * tk + kk, n = 32 * tn + nn;
    if (k >= K || n >= N) return;
    float g = 0.f;
    for (int s = 0; s < S; ++s) g += part[s][kk][at(kk, nn)];
    const int64_t i = mlp_offW_d(l) + (int64_t)k * N + n;
    if (!ADAM) {
        u.g[i] = g;
        return;
    }
    const uint16_t h = f2bf(mlp_adam(u, i, g));
    if (l == 0) {
        u.W[MLP_WB0 + (int64_t)((n >> 4) * 64 + (n & 15) + 16 * (k >> 2)) * 4 + (k & 3)] = h;
    } else if (l < 4) {
        u.W[MLP_WB1 + (int64_t)(l - 1) * 65536 + mlp_frag(k, n, 8)] = h;
        u.W[MLP_WT1 + (int64_t)(l - 1) * 65536 + mlp_frag(n, k, 8)] = h;
    } else {
        u.W[MLP_WB4 + mlp_frag(k, n, 8)] = h;
        u.W[MLP_WT4 + mlp_frag(n, k, 2)] = h;
    }
}

int64_t mlp_pack_count() { return MLP_WPK; }

hipError_t launch_mlp_pack(const float* P, uint16_t* W, hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_pack, dim3((unsigned)((MLP_WPK + 255) / 256)), dim3(256), 0, st, P, W);
    return hipGetLastError();
}

hipError_t launch_mlp_step(const MlpStep& a, hipStream_t st)
{
    if (a.rt == 1)
        hipLaunchKernelGGL(k_mlp_step<1>, dim3((unsigned)(a.Mpad / 16)), dim3(1024), 0, st, a);
    else
        hipLaunchKernelGGL(k_mlp_step<2>, dim3((unsigned)(a.Mpad / 32)), dim3(1024), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_mlp_update(bool adam, const MlpUpdate& u, hipStream_t st)
{
    const dim3 grid(MLP_UT + MLP_UB + 1);
    if (adam)
        hipLaunchKernelGGL(k_mlp_update<true>, grid, dim3(1024), 0, st, u);
    else
        hipLaunchKernelGGL(k_mlp_update<false>, grid, dim3(1024), 0, st, u);
    return hipGetLastError();
}

int64_t mlp_w16_count() { return MLP_W16_TOTAL; }

hipError_t launch_pack_w16(const float* P, uint16_t* W16, hipStream_t st)
{
    hipLaunchKernelGGL(k_pack_w16, dim3((unsigned)((MLP_W16_TOTAL + 255) / 256)), dim3(256), 0, st, P, W16);
    return hipGetLastError();
}

hipError_t launch_mlp_fused(int mode, int64_t M, const float* X, const uint16_t* W16, const float* P, float* Y,
                            const float* out_mu, const float* out_sd, const float* obs, int n_sum, float tol,
                            float* dist, uint8_t* keep, hipStream_t st)
{
    if (M <= 0) return hipSuccess;
    const dim3 grid((unsigned)((M + MLP_RT - 1) / MLP_RT));
    if (mode == 0)
        hipLaunchKernelGGL(k_mlp_fused<0>, grid, dim3(256), 0, st, M, X, W16, P, Y, out_mu, out_sd, obs, n_sum, tol, dist,
                           keep);
    else
        hipLaunchKernelGGL(k_mlp_fused<1>, grid, dim3(256), 0, st, M, X, W16, P, Y, out_mu, out_sd, obs, n_sum, tol, dist,
                           keep);
    return hipGetLastError();
}

}  // namespace swim
