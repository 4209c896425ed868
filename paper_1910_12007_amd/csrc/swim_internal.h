// swim_internal.h -- host-side interface between the C ABI (swim_capi.hip)
// and the kernel launchers (swim_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "swim_math.h"

namespace swim {

// Layout of a batch of independent systems (one hydrodynamic domain each),
// all device pointers indexed by the system id s.  System s holds nswim[s]
// filaments of npt[s] points; its filaments are [sw_off[s], sw_off[s+1]) of
// the parameter table; pt_off[s] is the start of its points in the
// large-system position buffers (unused by the persistent kernel).
struct Batch {
    int64_t n_sys;
    const int64_t* pt_off;
    const int64_t* sw_off;
    const int32_t* npt;      // points per filament
    const int32_t* nswim;    // filaments per system
    const double* params;    // [n_filaments][9]
    const void* sysc;        // SysConst<T>[n_sys]
    const void* sysc64;      // SysConst<double>[n_sys] (FP32 runs: builds the kernel tables)
    const void* tab;         // kernel tables: TabSys[n_sys] (FP32), TabSys64[n_sys] (FP64)
    int32_t alone;           // FP32 persistent runs: no more workgroups than compute units
};

struct Run {
    int32_t steps;
    double dt;
    int32_t obs_every;
    int32_t n_obs;
    double eps_over_ds;
    // early rejection against a known tolerance (persistent kernel, one
    // swimmer per system): with stop_data ([n_obs][2] head data) set, a run
    // stops with SWIM_ST_REJECTED_ once the running sum of its squared head
    // deviations exceeds stop_ssq (the sum only grows, so its final
    // distance exceeds the tolerance)
    const double* stop_data = nullptr;
    double stop_ssq = 0.0;
};

// all launchers return hipError_t of the launch
// (dtype 0 also writes the FP64 constants into sysc64, for the kernel tables)
// blob: 0 the kernel reading's blob, 1 the paper's blob (closed forms at
// alpha = 0, quadrature for alpha > 0)
// whether a launch fits: a grid of 2^32 threads and more is cut short without an
// error
inline bool grid_fits(int64_t blocks, int threads)
{
    return blocks <= 0x7FFFFFFF && blocks * threads < ((int64_t)1 << 32);
}
hipError_t launch_sysconst_batch(int dtype, int64_t n_sys, const int64_t* sw_off, const int32_t* npt,
                                 const double* params, double eps_over_ds, void* sysc, void* sysc64,
                                 int32_t* status, int blob, hipStream_t st);
hipError_t launch_sysconst(int dtype, int64_t n_sys, const double* alpha, const double* eps,
                           void* sysc, void* sysc64, int blob, hipStream_t st);
// blk0: first 64-target workgroup of each system (prefix, n_sys + 1), nb their number
hipError_t launch_pair_velocity(int dtype, int64_t n_sys, int64_t nb, const int64_t* blk0, const int64_t* pt_off,
                                const void* sysc, const void* tab, const void* x, const void* y, const void* fx,
                                const void* fy, void* ux, void* uy, hipStream_t st);
// FP32 systems of ORDERED_MIN points and more, one-sided, with the bits of the
// tile pairs (launch_tile_velocity)
constexpr int ORDERED_MIN = 512;
hipError_t launch_ordered_velocity(int64_t n_sys, int64_t nb, const int64_t* blk0, const int64_t* pt_off,
                                   const void* sysc, const void* tab, const void* x, const void* y, const void* fx,
                                   const void* fy, void* ux, void* uy, hipStream_t st);
// bytes of one system's kernel table (TabSys, TabSys64)
size_t table_bytes(int dtype);
// FP64 velocity sums evaluate systems of at most this many points directly where
// the kernel functions are closed forms (all but the paper's blob at alpha > 0)
constexpr int DIRECT64_MAX = 24;
static_assert(DIRECT64_MAX <= 64, "one workgroup of 64 targets per system");
hipError_t launch_direct_velocity(int64_t n_sys, int64_t nb, const int64_t* blk0, const int64_t* pt_off,
                                  const void* sysc, const void* x, const void* y, const void* fx, const void* fy,
                                  void* ux, void* uy, hipStream_t st);
// kernel tables of systems [s0, s0 + n) (FP64 constants sysc64) into tab[s];
// pt_off, if not null: FP64, without those of the systems evaluated directly
hipError_t launch_table_build(int dtype, int64_t s0, int64_t n, const void* sysc64, void* tab, int blob, hipStream_t st,
                              const int64_t* pt_off = nullptr);
hipError_t launch_forces(int dtype, int64_t n_fil, const int64_t* fil_off, const int32_t* npt,
                         const double* params, double t, const void* x, const void* y, void* fx,
                         void* fy, hipStream_t st);
// persistent forward run, one workgroup of wps wavefronts per system
// (systems of at most 64*tpl points; tpl in {1,2,3,4,6,8}, wps in {1,2,4})
hipError_t launch_forward(int dtype, int tpl, int wps, int n_blocks, const Batch& b,
                          const Run& r, const int32_t* order, int32_t* queue, void* obs,
                          void* speed, int32_t* status, int32_t* steps_done, hipStream_t st);
// queue order of some buckets (segments of the order array, at most
// ORDER_MAX systems each): long runs first
constexpr int ORDER_SEGS = 6, ORDER_MAX = 262144;
struct OrderSegs {
    int64_t start[ORDER_SEGS];
    int32_t count[ORDER_SEGS];
};
hipError_t launch_order_runs(int n_seg, const OrderSegs& seg, const int32_t* in, const int64_t* sw_off,
                             const int32_t* npt, const double* params, double dt, int32_t* out, hipStream_t st);
// smallest waves per system of the persistent kernel for tpl targets per lane
int forward_min_wps(int tpl);
size_t forward_lds_bytes(int dtype, int tpl, int wps);
// set the kernels' dynamic-LDS limits ahead of launches (needed before a
// stream capture, in which the launch itself must not change attributes)
hipError_t prepare_forward(int dtype, int tpl, int wps);
hipError_t prepare_big_step(int dtype, int tpl, int32_t max_pts);
int forward_blocks_per_cu(int dtype, int tpl, int wps);
// one forward-Euler step of large systems, targets split over workgroups
struct BigState {
    void* xh[2];   // position hi parts, double-buffered, [n_points] T
    void* yh[2];
    void* xl[2];   // lo parts
    void* yl[2];
    void* head0;   // [n_filaments][2] T, initial head positions
};
// the symmetric FP32 tile-pair path: the systems that take it, cut into
// tiles of BIG_TILE_POINTS points, every pair of tiles one workgroup
constexpr int BIG_TILE_POINTS = 128;
struct BigTiles {
    int64_t n_big, n_pairs, n_tiles;  // systems, tile pairs and tiles of all of them
    const int64_t* list;   // [n_big] system
    const int64_t* off0;   // [n_big + 1] first off-diagonal tile pair
    const int64_t* tile0;  // [n_big + 1] first tile
    const int64_t* slot0;  // [n_big] first partial slot (nt * nt slots)
    const int64_t* pt0;    // [n_big] first point
    const int32_t* cnt;    // [n_big] points
    void* part;            // slots of one double pair per point: slot t * nt + q = tile t's sums over tile q
    void* src;             // forward runs: sources of all points (position, force)
};
// velocities for given forces
hipError_t launch_tile_velocity(const BigTiles& bt, const void* sysc, const void* tab, const void* x, const void* y,
                                const void* fx, const void* fy, void* ux, void* uy, hipStream_t st);
// forward steps: the first step's sources, then tile pairs and the update
hipError_t prepare_big_pairs();
hipError_t launch_big_sources(const BigTiles& bt, const Batch& b, const BigState& s, hipStream_t st);
hipError_t launch_big_sym_step(const BigTiles& bt, const Batch& b, const BigState& s, int step, const Run& r, void* obs,
                               int32_t* status, int32_t* steps_done, hipStream_t st);
hipError_t launch_big_init(int dtype, const int64_t* list, int64_t n_list, const Batch& b,
                           const BigState& s, int32_t* status, void* obs, int32_t n_obs,
                           hipStream_t st);
hipError_t launch_big_step(int dtype, int tpl, int64_t n_blocks, const int64_t* blk_sys,
                           const int64_t* blk_first, int32_t max_pts, const Batch& b,
                           const BigState& s, int step, const Run& r, void* obs, int32_t* status,
                           int32_t* steps_done, hipStream_t st);
hipError_t launch_big_finish(int dtype, const int64_t* list, int64_t n_list, const Batch& b,
                             const BigState& s, int buf, const Run& r, void* speed,
                             const int32_t* status, int32_t* steps_done, hipStream_t st);
size_t big_step_lds_bytes(int dtype, int32_t max_pts);

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st);
hipError_t launch_abc_distance(int dtype, int64_t n, int32_t n_obs, const void* obs,
                               const double* data, const int32_t* status, double* dist,
                               hipStream_t st);
// k-th smallest (1-based) of n doubles -> *out (device); single workgroup radix select
hipError_t launch_select_kth(int64_t n, const double* v, double q, double* out, hipStream_t st);
hipError_t launch_accept(int64_t n, const double* dist, const double* tol, uint8_t* acc,
                         hipStream_t st);
hipError_t launch_gauss_loglik(int dtype, int64_t n, int32_t n_obs, const void* obs, const double* data,
                               const double* sigma, const int32_t* status, double* logl, hipStream_t st);

// surrogate MLP (swim_mlp.hip)
// one training step (swim_mlp.hip): rows through the network and back ...
constexpr int MLP_DBN = 4 * 256 + 33;  // biases: hidden layers, then the outputs
struct MlpStep {
    const float *X, *T;         // [nrows][5], [nrows][33]
    const int32_t* perm;        // rows of the batch (null: 0..M-1); an index outside [0, nrows) gives a NaN row
    int64_t nrows, M, Mpad;     // rows of X and T, of the batch, the batch padded to 32
    const float* P;             // parameters (the biases are read)
    const uint16_t* W;          // packed bfloat16 weights (launch_mlp_pack)
    uint16_t *XT, *HT, *DT, *YT;  // feature-major bfloat16 [16], [4][256], [4][256], [48] x Mpad
    float* DF;                  // gradients in FP32, feature-major [MLP_DBN] x Mpad
    float* lossp;               // squared errors [3] per workgroup
    float sc;                   // 2 / (33 M)
    int kf, ko, kb, kb4;        // 32-wide pieces per slice of the sums: hidden, output, back, back from the output
    int rt;                     // 16-row tiles per workgroup (1 or 2)
};
// ... then weight gradients with Adam (or into g)
struct MlpUpdate {
    int64_t M, Mpad, nwg;       // nwg: workgroups of the step
    const uint16_t *XT, *HT, *DT, *YT;
    const float *DF, *lossp;
    float *p, *m, *v, *g, *loss;  // loss may be null
    uint16_t* W;
    int kw, kw4, kw0;           // 32-row pieces per slice: hidden layers, output, input
    float lr, b1, b2, c1, c2, eps;
};
int64_t mlp_pack_count();
hipError_t launch_mlp_pack(const float* P, uint16_t* W, hipStream_t st);
hipError_t launch_mlp_step(const MlpStep& a, hipStream_t st);
hipError_t launch_mlp_update(bool adam, const MlpUpdate& u, hipStream_t st);
hipError_t launch_compact(int64_t n, const uint8_t* keep, int32_t* counts, int64_t* idx,
                          int64_t* total, hipStream_t st);
hipError_t launch_features(int64_t n, const double* theta, double b, double om, const float* mu,
                           const float* sd, float* X, hipStream_t st);
hipError_t launch_targets(int dtype, int64_t n, int n_obs, const void* obs, const void* speed,
                          double x0, double y0, const int32_t* idx, int n_sum, float* T,
                          hipStream_t st);
hipError_t launch_colstats(int64_t n, int cols, const float* A, float* mu, float* sd, hipStream_t st);
hipError_t launch_standardize(int64_t n, int cols, float* A, const float* mu, const float* sd,
                              hipStream_t st);
hipError_t launch_prior_draw(uint64_t seed, int64_t n, const double* lo, const double* hi,
                             double* theta, hipStream_t st);
hipError_t launch_param_rows(int64_t cap, const int64_t* n_dev, const int64_t* idx, int64_t n_theta,
                             const double* theta, double b, double om, double kw, double* rows,
                             hipStream_t st);
hipError_t launch_gather_f32(int64_t cap, const int64_t* n_dev, const int64_t* idx, int64_t n_src,
                             const float* src, int cols, float* dst, hipStream_t st);
hipError_t launch_flag_eq(int64_t n, const int32_t* v, int32_t want, uint8_t* keep, hipStream_t st);
hipError_t launch_flag_bounded(int64_t n, const float* T, int nt, int n_disp, float max_disp, uint8_t* keep,
                               hipStream_t st);

// fused MLP inference (mode 0: outputs Y[M][33]; mode 1: prescreen distance
// and keep flag), from the bfloat16 weight copy W16 (launch_pack_w16)
int64_t mlp_w16_count();
hipError_t launch_pack_w16(const float* P, uint16_t* W16, hipStream_t st);
hipError_t launch_mlp_fused(int mode, int64_t M, const float* X, const uint16_t* W16, const float* P, float* Y,
                            const float* out_mu, const float* out_sd, const float* obs, int n_sum, float tol,
                            float* dist, uint8_t* keep, hipStream_t st);

// full sperm model (swim_sperm.hip): shape shared by all systems of a call
struct SpermShape {
    int32_t nf, nh, nsw, pad;   // flagellum points, head points, swimmers per system
    double ds, ch, hr, dn, dth; // 1/(nf-1), head chord, head radius, neck gap, 2 pi/nh
    double eps;                 // blob width
    double L0[5];               // neck rest lengths (last flagellum point to pi-dth, pi,
                                // pi+dth; the one before to pi-dth, pi+dth)
};
struct SpermRun {
    int64_t n_sys;
    const double* sysp;  // [n_sys][SWIM_SP_NPARAM]
    const double* swp;   // [n_sys * nsw][3]: x0, y0, phase
    int32_t steps, obs_every, n_obs;
    int32_t oct;         // octaves of the table that a system keeps in LDS (FP64: all or none)
    double dt;
};
hipError_t launch_sperm_setup(int dtype, int64_t n_sys, int32_t nsw, double eps, const double* sysp,
                              const double* swp, void* sysc, void* sysc64, int32_t* status, int blob,
                              hipStream_t st);
hipError_t prepare_sperm(int dtype, int tpl, int wps);
// FP32 octaves in LDS: the whole table, or the first
constexpr int SPERM_OCT_ALL = 44, SPERM_OCT_HEAD = 24;
// FP64 shapes with a second build that holds the whole table in LDS (SpermRun::oct != 0)
constexpr bool sperm_lds64(int dtype, int tpl, int wps) { return dtype == 1 && tpl <= 4 && wps == 8; }
int sperm_blocks_per_cu(int dtype, int tpl, int wps, const SpermShape& g, int oct);
// persistent run, one workgroup of wps wavefronts per system (tpl in
// {1,2,3,4,6,8}, wps in {2,4,8})
hipError_t launch_sperm_forward(int dtype, int tpl, int wps, int nblocks, const SpermShape& g, const SpermRun& r,
                                const void* sysc, const void* tabs, int32_t* queue, void* head, void* tail,
                                int32_t* status, hipStream_t st);
// observables per system and sample k = 1..n_obs into g[n_sys][n_obs][2]:
// kind 0 head-centre velocity of swimmer 0, kind 1 (tail, head) distances of
// swimmers 0 and 1
hipError_t launch_sperm_observables(int dtype, int kind, int64_t n_sys, int32_t nsw, int32_t n_obs, double dt_obs,
                                    const void* head, const void* tail, const int32_t* status, double* g,
                                    hipStream_t st);
// Gaussian log-likelihood with standard deviations sig2[i][0] (entries 0,
// 2, ...) and sig2[i][1] (entries 1, 3, ...); status may be NULL
hipError_t launch_gauss_loglik2(int64_t n, int32_t n_obs, const double* g, const double* data, const double* sig2,
                                const int32_t* status, double* logl, hipStream_t st);

// velocity and pressure at arbitrary points (swim_field.hip): constants of one
// fluid and blob.  The pressure weight m(r) / (2 pi r^2) is inv_2pi / R^2
// (stokes), the power series ser[] in delta = r^2/eps^2 for delta < 1/4, and
// inv_2pi (1 - eps K1(alpha R) / (R K1e)) / r^2 otherwise.
constexpr int FIELD_NSER = 26;
struct FieldConst {
    SysConst<float> c32;
    SysConst<double> c64;
    double h1c, inv_e2, e2, eps, alpha, K1e, inv_2pi;
    int32_t stokes, paper;  // paper: the paper's blob (mass 1 - eps^3/R^3)
    double ser[FIELD_NSER];
};
// whether an FP64 field evaluates its pairs directly instead of from a table
bool field_direct64(const FieldConst& fc, int64_t n);
// FP32: fc_dev (fc in device memory), tab and wtab; FP64: tab, or null for direct evaluation
hipError_t launch_flow_field(int dtype, int64_t n, const void* x, const void* y, const void* fx, const void* fy,
                             const FieldConst& fc, const FieldConst* fc_dev, int64_t nt, const void* tx, const void* ty,
                             void* u, void* v, void* p, const void* tab, void* wtab, hipStream_t st);

}  // namespace swim
