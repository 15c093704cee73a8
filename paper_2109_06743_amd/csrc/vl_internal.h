// Internal interface between the C ABI (vl_api.hip) and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/vl.h"
#include "vl_common.h"

namespace vl {

struct VGridArgs {
    int nv[3];
    double lo[3], dv[3];
    double m;
};

struct V3Params;  // pfc_kernels.hip

// Where a kernel leaves the maximum of its output.  A slot holds kSlotMax
// entries of 8 bytes: up to `direct` per-block maxima stay in the slot for the
// consumer's waves to fold (max_of; a launch saved), more go to part and are
// reduced into the slot's first entry.  kDirectX where the X operator consumes
// them: its waves are few and walk many cells (1024 partials: two batches of
// loads).  kDirectV where the velocity operator does: every cell's waves fold
// them again (1024 partials cost it 20 % at 256x128x16^3, 64 nothing).
// slot null: no maximum wanted.  *n receives the number of entries the slot
// holds; with `fixed` set that number whatever the launch's blocks, the producer
// filling up with zeros (a maximum kept for the next step, which may be part of a
// graph, must not depend on dt).
constexpr int kSlotMax = 1024;
constexpr int kDirectX = 1024, kDirectV = 64;
struct MaxSink {
    void* slot = nullptr;
    void* part = nullptr;
    int* n = nullptr;
    int most = 0;
    int fixed = 0;
    bool direct(long long blocks) const { return blocks <= most; }
    template <class T>
    typename Bits<T>::U* target(long long blocks) const {
        if (!slot) return nullptr;
        *n = direct(blocks) ? (fixed ? fixed : (int)blocks) : 1;
        return (typename Bits<T>::U*)(direct(blocks) ? slot : part);
    }
};

template <class T>
hipError_t launch_pfc_x(const T* fin, T* fout, int rows, int nx, long long Nv, int inner, double vx_lo, double dvx,
                        double tau_dx, MaxRef finf, const MaxSink& sink, hipStream_t st);
// g (the Poisson table) set: E is formed from the densities of mom and stored
// to E; null: E is read.
template <class T>
hipError_t launch_pfc_v1(const T* fin, T* fout, int nx, int nv, double* E, const double* mom, const double* g,
                         double q, double qm_tau_dv, MaxRef finf, const MaxSink& sink, hipStream_t st);
struct V3Params {
    int nvx, nvy, nvz;
    double lo[3], dv[3], inv_dv[3];
    double qm, tau;
    float inv_nvz, inv_nvy;   // 1/nvz, 1/nvy, for the exact row index (e + 0.5) / nvz of small e
};

// Row index e / n for 0 <= e < 2^16 without integer division: (e + 0.5)/n is
// at least 1/(2n) away from an integer, while the float product is off by at
// most 2^16/n * 2^-23 < 1/(2n).
__device__ __forceinline__ int row_of(int e, float inv_n) { return (int)(((float)e + 0.5f) * inv_n); }
template <class T>
hipError_t launch_pfc_v3(const T* fin, T* fout, long long cells, const double* E, const double* B, const V3Params& P,
                         MaxRef finf, const MaxSink& sink, hipStream_t st);
// Threads per block of the general kernels whose threads own pencils.
int pencil_threads(const int* pens, int n, size_t lds, int cap, long long cells, bool wide);
size_t v3_shared_bytes(int nvx, int nvy, int nvz, size_t elem);
// V(tau) by the backsubstitution split: three affine sweeps with per-face
// feet (every velocity axis <= 32).
template <class T>
hipError_t launch_pfc_v3b(const T* fin, T* fout, long long cells, const double* E, const double* B, const V3Params& P,
                          MaxRef finf, const MaxSink& sink, hipStream_t st);
template <class T>
hipError_t launch_array_max(const T* f, long long n, const MaxSink& sink, hipStream_t st);
// Launchers that produce a maximum leave it as their sink says: few per-block
// maxima in the slot itself, for the consumer to fold; more in `part` (8 bytes
// per block of their grid), which they fold into the slot in another launch --
// but for launch_fit3, whose partials launch_fit_fold folds.  These give the
// grid sizes, to size `part`.
long long pfc_x_blocks(int rows, int nx, long long Nv);
long long pfc_xy_blocks(int nx, int ny, int nvx, int nvy, int nvz);
// Fused X(tau) of 2X3V (x then y sweep, one f_inf); fout must not alias fin.
// per = 0: reflecting y walls, 1: periodic y.
template <class T>
hipError_t launch_pfc_xy(const T* fin, T* fout, int nx, int ny, int nvx, int nvy, int nvz, double vx_lo, double dvx,
                         double tau_dx, double vy_lo, double dvy, double tau_dy, int per, MaxRef finf,
                         const MaxSink& sink, hipStream_t st);
constexpr long long kMaxArrayBlocks = 2048;
// Reductions of up to kFoldOne per-block partials (maxima, clip counts) run in
// one launch of one block, longer ones in two:
// fin_split(n).blocks <= kFinStage blocks fold ranges of fin_split(n).chunk
// partials into a stage of kFinStage entries that sits fin_stage(n, size)
// bytes after the partials' start, then one wave folds the stage.  A partials
// buffer of n entries of `size` bytes therefore needs kFinSlack bytes beyond
// its n * size.
constexpr long long kFoldOne = 65536;
constexpr int kFinStage = 64;
constexpr long long kFinRange = 8192;          // partials per first-level block, at least
constexpr size_t kFinSlack = 128 + kFinStage * 8;
struct FinSplit {
    int blocks;
    long long chunk;
};
inline FinSplit fin_split(long long n) {
    long long g = (n + kFinRange - 1) / kFinRange;
    g = g < 1 ? 1 : (g > kFinStage ? kFinStage : g);
    return {(int)g, (n + g - 1) / g};
}
__host__ __device__ inline size_t fin_stage(long long n, size_t size) { return ((size_t)n * size + 127) / 128 * 128; }
template <class T>
hipError_t launch_max_finalize(const void* part, long long n, void* slot, hipStream_t st);

template <class T>
hipError_t launch_moments3(const T* f, double* mom, long long cells, const VGridArgs& a, hipStream_t st);
template <class T>
hipError_t launch_moments1(const T* f, double* mom, long long cells, int nv, double vlo, double dv, double m,
                           hipStream_t st);
// Edge of the large cubic velocity grid with fixed-size kernels (FP32 only:
// 34 x 34 x 35 floats = 161840 bytes of LDS per cell in the V operator).
constexpr int kBigCube = 34;
// Per-cell parameters of the fits, kFitCellDoubles doubles per spatial cell of
// device scratch: launch_fit3_params fills those of ns species (one after the
// other) and rescales U in place, then launch_fit3 runs per species.
constexpr int kFitCellDoubles = 20;
template <class T>
hipError_t launch_fit3_params(int ns, const double* const* mom_pre, double* const* U, const VGridArgs* a,
                              long long cells, double* params, void* counters, hipStream_t st);
template <class T>
hipError_t launch_fit3(const T* fin, T* fout, double* mom_post, void* counters, long long cells, const VGridArgs& a,
                       const MaxSink& sink, unsigned* clip_part, const double* params, hipStream_t st);
// launch_fit3 leaves per-block maxima in the sink and per-cell clip counts in
// clip_part; launch_fit_fold, after the fits of all ns species, folds them
// into the sinks' slots and the counters.  Until then a slot is valid only
// where its sink is direct for that many cells.
template <class T>
hipError_t launch_fit_fold(int ns, const MaxSink* sinks, unsigned* const* clips, void* counters, long long cells,
                           hipStream_t st);
template <class T>
hipError_t launch_fit1(const T* fin, T* fout, const double* mom_pre, const double* Uin, double* U, double* mom_post, void* counters,
                       long long cells, int nv, double vlo, double dv, double m, const MaxSink& sink,
                       hipStream_t st);

// Green's function of the 1X1V Poisson solver, g[N], and the solve with it.
hipError_t launch_poisson_green(int N, double L, double* g, hipStream_t st);
hipError_t launch_poisson(const double* mom, int N, double q, const double* g, double* E, hipStream_t st);
// mom[s]: per-cell records of mstride doubles holding n u at offsets 1..3
// (raw moments: 20; fluid state: 10).
hipError_t launch_maxwell_half(double* yee, int nx, int ny, const double* const* mom, const double* q, int ns,
                               double dt, double c, double dx, double dy, hipStream_t st, int mstride = 20,
                               int per = 0);
hipError_t launch_cell_fields(const double* yee, int nx, int ny, double* E, double* B, hipStream_t st);
hipError_t launch_field_energy(const double* fields, int dim_x, int nx, int ny, double c, double dX, double* part,
                               double* out, hipStream_t st);
// The same half step out of place (from and to must not overlap), in one
// launch, with the cell-centred averages of the fields before (at_from) and
// after (at_to) and 2 after - before (ahead); null pointers: not wanted (ahead
// needs the other two).
struct CellFields {
    double* E = nullptr;
    double* B = nullptr;
};
hipError_t launch_yee_half(const double* from, double* to, int nx, int ny, const double* const* mom, const double* q,
                           int ns, double dt, double c, double dx, double dy, int mstride, int per,
                           const CellFields& at_from, const CellFields& at_to, const CellFields& ahead,
                           hipStream_t st);

// Per-species operands of one fluid stage: up to two species per launch.
struct FluidSet {
    const double* Us[2];          // stage state; U_out must not be it
    const double* Un[2];          // state of the step's start (U_out may be it)
    double* Uo[2];
    const double* QA[2];          // kinetic third moments (raw-moment layout)
    const double* QB[2];
    const float* y[2];            // network outputs [cells][16] and scales [cells]
    const double* scale[2];
    const int* fallback[2];       // network: take the kinetic moment where set (may be null)
    double m[2], q[2], gchi[2];
};
// Third moment of a stage: wa QA + wb QB; that of zero heat flux plus the Eq. 5
// source of P (gchi = chi / k0); that of the network's heat flux.
enum { kThirdFromF = 0, kThirdGradient = 1, kThirdNetwork = 2 };

// Scratch of one species' SSP-RK3 step of the 3V fluid (doubles): U1, U2.
inline size_t fluid_rk3_3v_doubles(int nx, int ny) { return 20 * (size_t)nx * ny; }

// State buffers of stage k (0..2) of species s: U -> U1 -> U2 -> U.
inline void rk3_buffers(FluidSet& S, int s, int k, double* U, double* work, long long cells) {
    double* U1 = work;
    double* U2 = U1 + cells * 10;
    S.Us[s] = k == 0 ? U : (k == 1 ? U1 : U2);
    S.Un[s] = U;
    S.Uo[s] = k == 0 ? U1 : (k == 1 ? U2 : U);
}

// One SSP-RK3 step of ns (1 or 2) species, each stage launched once for all
// of them; work: ns * fluid_rk3_3v_doubles(nx, ny) doubles.
hipError_t launch_fluid_rk3_3v_set(int ns, double* const* U, const double* const* mom_t, const double* const* mom_t1,
                                   const double* E_t, const double* B_t, const double* E_t1, const double* B_t1,
                                   const double* E_th, const double* B_th, double dt, int nx, int ny, const double* q,
                                   const double* m, double dx, double dy, double* work, hipStream_t st, int per);
// One stage (0..2) of the step for ns species.
hipError_t launch_fluid_stage_3v_set(const FluidSet& S, int ns, int third, int stage, double wa, double wb,
                                     const double* E, const double* B, double dt, int nx, int ny, double dx,
                                     double dy, hipStream_t st, int per);
// U -> Uout (which may be U; work: 3 nx doubles, used then).  g set: the stage
// fields are the Poisson solves of mom_t, mom_t1 and their mean.
hipError_t launch_fluid_rk3_1v(double* U, double* Uout, const double* mom_t, const double* mom_t1, const double* E_t,
                               const double* E_t1, const double* E_th, const double* g, double dt, int nx, double q,
                               double m, double dx, double* work, hipStream_t st);

// learned heat-flux closure (mlp_kernels.hip)
constexpr int kMlpParams = 13520;
// Per-species operands of the network kernels for up to two species per
// launch; the features, scales and outputs of the set's species are stored
// one after the other (cells of species 0, then 1).
struct MlpSet {
    const double* M[2];     // features and judge: moment (stride 20) or fluid (stride 10) records
    int* fallback[2];       // judge output
    double* err[2];         // judge output
    double m[2];
};
hipError_t launch_mlp_features_set(const MlpSet& S, int ns, int s0, int stride, const double* B, int nx, int ny,
                                   unsigned short* x, double* scale, hipStream_t st);
// Features and network in one launch: outputs y [cells][16] and scales.
hipError_t launch_mlp_network_set(const MlpSet& S, int ns, int s0, int stride, const double* B, int nx, int ny,
                                  const float* params, double* scale, float* y, hipStream_t st);
hipError_t launch_mlp_judge_set(const MlpSet& S, int ns, const double* scale, const float* y, long long cells,
                                double tol, double* part, hipStream_t st);
hipError_t launch_mlp_features(const double* M, int stride, const double* B, int nx, int ny, double m, int species,
                               unsigned short* x, double* scale, hipStream_t st);
hipError_t launch_mlp_targets(const double* M, long long cells, double m, float* y, hipStream_t st);
hipError_t launch_mlp_forward(const float* P, const unsigned short* x, long long n, float* y, hipStream_t st);
size_t mlp_grad_blocks(long long n);
size_t mlp_part_floats(long long n);
hipError_t launch_mlp_gradient(const float* P, const unsigned short* x, const float* t, long long n, float* part,
                               float* grad, hipStream_t st,
                               const long long* idx = nullptr, long long nrows = 0);
// gradient (as launch_mlp_gradient) and the Adam update of step `step`, fused
// into the gradient sum
hipError_t launch_mlp_train_step(float* P, float* m1, float* m2, long long step, double lr,
                                 const unsigned short* x, const float* t, long long n, float* part, float* grad,
                                 hipStream_t st, const long long* idx = nullptr, long long nrows = 0);
size_t mlp_judge_part_doubles();

template <class T>
hipError_t launch_mass_energy(const T* f, const double* mom, long long cells, long long nv, int kmom, int dimv,
                              double dV, double dX, double* out, double* part, hipStream_t st);

}  // namespace vl
