// Velocity moments and moment fitting for gfx950.
//
// Moments (Sec. 2.1 of arXiv 2109.06743, definitions after Eq. 1), midpoint
// rule on the velocity cell centres, accumulated in FP64 whatever the storage
// type of f.  3V sums are separable: each thread forms the four row sums
// sum_z f v_z^k (k = 0..3) of one (v_x, v_y) row, then the row's share of the
// 20 raw moments needs 20 FP64 operations per row instead of per cell.
//
// Moment fitting (Algorithm 1, "Moment Fitting"; Sec. 2.2): per cell
//   f' = f - M[n_V, u_V, T_V] + M[n_V, u_F, T_F],  f'' = max(f', 0),
//   f_new = f'' n_V / (sum f'' dV),
// M the ten-moment Maxwellian n g / (sum g dV), g = exp(-(m/2) w^T T^-1 w),
// w = v - u.  Exponentials and f in the storage type; quadratic-form
// coefficients, normalisation sums, the rescale factor and all moments FP64.
#include "vl_internal.h"

namespace vl {

struct VGrid {
    int nvx, nvy, nvz;
    double lo[3], dv[3];
    double m;
    float inv_nvz;
};

__device__ __forceinline__ double vc(const VGrid& G, int d, int i) { return G.lo[d] + (i + 0.5) * G.dv[d]; }

template <class T>
__global__ void __launch_bounds__(256) moments1_kernel(const T* __restrict__ f, double* __restrict__ mom, int nv,
                                                       double vlo, double dv, double mass) {
    __shared__ double red[4 * 4];
    const long long cell = blockIdx.x;
    const T* src = f + cell * nv;
    double acc[4] = {0, 0, 0, 0};
    for (int j = threadIdx.x; j < nv; j += blockDim.x) {
        const double v = vlo + (j + 0.5) * dv;
        const double x = (double)src[j];
        const double xv = x * v;
        acc[0] += x;
        acc[1] += xv;
        acc[2] += xv * v;
        acc[3] += xv * v * v;
    }
    block_sum<4>(acc, red);
    if (threadIdx.x == 0) {
        mom[cell * 4 + 0] = acc[0] * dv;
        mom[cell * 4 + 1] = acc[1] * dv;
        mom[cell * 4 + 2] = mass * acc[2] * dv;
        mom[cell * 4 + 3] = mass * acc[3] * dv;
    }
}

// ------------------------------------------------------------------ fit ----
// Symmetric 3x3 stored as (xx, xy, xz, yy, yz, zz).  Returns false unless the
// matrix is positive definite (Cholesky pivots > 0); inv receives its inverse.
__device__ __forceinline__ bool spd_inverse(const double (&a)[6], double (&inv)[6]) {
    const double l11sq = a[0];
    if (!(l11sq > 0.0)) return false;
    const double l11 = sqrt(l11sq);
    const double l21 = a[1] / l11, l31 = a[2] / l11;
    const double l22sq = a[3] - l21 * l21;
    if (!(l22sq > 0.0)) return false;
    const double l22 = sqrt(l22sq);
    const double l32 = (a[4] - l31 * l21) / l22;
    const double l33sq = a[5] - l31 * l31 - l32 * l32;
    if (!(l33sq > 0.0)) return false;
    // inverse via cofactors (the matrix is SPD, so det > 0)
    const double c00 = a[3] * a[5] - a[4] * a[4];
    const double c01 = a[2] * a[4] - a[1] * a[5];
    const double c02 = a[1] * a[4] - a[2] * a[3];
    const double c11 = a[0] * a[5] - a[2] * a[2];
    const double c12 = a[1] * a[2] - a[0] * a[4];
    const double c22 = a[0] * a[3] - a[1] * a[1];
    const double det = a[0] * c00 + a[1] * c01 + a[2] * c02;
    const double id = 1.0 / det;
    inv[0] = c00 * id; inv[1] = c01 * id; inv[2] = c02 * id;
    inv[3] = c11 * id; inv[4] = c12 * id; inv[5] = c22 * id;
    return true;
}

// Mean velocity and temperature tensor from (n, nu, P) with T = (P - m n u u)/n.
__device__ __forceinline__ void u_and_T(const double* nuP, double n, double m, double (&u)[3], double (&T)[6]) {
    u[0] = nuP[0] / n; u[1] = nuP[1] / n; u[2] = nuP[2] / n;
    const int ia[6] = {0, 0, 0, 1, 1, 2}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int k = 0; k < 6; ++k) T[k] = (nuP[3 + k] - m * n * u[ia[k]] * u[ib[k]]) / n;
}

template <class T>
__device__ __forceinline__ T expo(T x);
template <> __device__ __forceinline__ float expo<float>(float x) { return __expf(x); }
template <> __device__ __forceinline__ double expo<double>(double x) { return exp(x); }

// ------------------------------------------------------- cubic blocks -------
// Velocity blocks with N cells per axis: thread t < N*N owns the v_x pencil at
// (v_y, v_z) = (t / N, t % N); element (ix, t) sits at t + N*N*ix, so the loads
// of a wave are contiguous and the only coordinate that varies along a thread's
// elements is v_x, which is uniform across the block (table in the arguments).
struct XTable {
    double v[kBigCube], v2[kBigCube], v3[kBigCube];
};

// The 20 raw moments as weighted sums of the pencil sums S_k = sum_x f v_x^k
// with the thread's transverse velocities (v_y, v_z).
__device__ __forceinline__ void pencil_moments(const double (&S)[4], double vy, double vz, double (&a)[20]) {
    const double vy2 = vy * vy, vz2 = vz * vz, vyz = vy * vz;
    a[0] = S[0];        a[1] = S[1];        a[2] = vy * S[0];   a[3] = vz * S[0];
    a[4] = S[2];        a[5] = vy * S[1];   a[6] = vz * S[1];
    a[7] = vy2 * S[0];  a[8] = vyz * S[0];  a[9] = vz2 * S[0];
    a[10] = S[3];       a[11] = vy * S[2];  a[12] = vz * S[2];  a[13] = vy2 * S[1];
    a[14] = vyz * S[1]; a[15] = vz2 * S[1]; a[16] = vy2 * vy * S[0];
    a[17] = vy2 * vz * S[0]; a[18] = vy * vz2 * S[0]; a[19] = vz2 * vz * S[0];
}

// Any velocity grid with axes up to 32: NW waves per cell (four cells per
// 256-thread block with NW = 1, for the small blocks), thread t owns the v_x
// pencils t, t + 64 NW, ... and reads them as they lie (unit stride over the
// lanes), in code for exactly their length, so that a pencil's loads are in
// flight together.  The kernel before took each cell through shared memory,
// one v_z row per thread: 100 x 50 cells of 20x16x24 FP32 124 us in a step;
// with eight loads in flight 69, this way 33 (4.6 TB/s).
template <class T, int N>
__device__ __forceinline__ void pencil_sums(const T* __restrict__ src, unsigned off, unsigned plane, const XTable& X,
                                            double (&S)[4]) {
    T v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = src[off + (unsigned)k * plane];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double g = (double)v[k];
        S[0] += g;
        S[1] = fma(g, X.v[k], S[1]);
        S[2] = fma(g, X.v2[k], S[2]);
        S[3] = fma(g, X.v3[k], S[3]);
    }
}

template <class T, int NW>
__global__ void __launch_bounds__(256)
moments3_kernel(const T* __restrict__ f, double* __restrict__ mom, long long cells, VGrid G, XTable X) {
    __shared__ double red[NW == 1 ? 1 : 4 * 20];
    __shared__ double fin_s[20];
    const int tid = threadIdx.x & (64 * NW - 1), lane = threadIdx.x & 63;
    const long long cell = NW == 1 ? (long long)xcd_work_index(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6)
                                   : (long long)xcd_work_index(blockIdx.x, gridDim.x);
    if (NW == 1 && cell >= cells) return;
    const int npen = G.nvy * G.nvz;
    const T* src = f + cell * npen * G.nvx;
    double acc[20];
#pragma unroll
    for (int q = 0; q < 20; ++q) acc[q] = 0.0;
    for (int t = tid; t < npen; t += 64 * NW) {
        double S[4] = {0.0, 0.0, 0.0, 0.0};
#define VL_LEN(N)                                                          \
    case N:                                                                \
        pencil_sums<T, N>(src, (unsigned)t, (unsigned)npen, X, S);         \
        break;
        VL_LENGTHS(G.nvx)
#undef VL_LEN
        const int iy = row_of(t, G.inv_nvz);
        double a[20];
        pencil_moments(S, vc(G, 1, iy), vc(G, 2, t - iy * G.nvz), a);
#pragma unroll
        for (int q = 0; q < 20; ++q) acc[q] += a[q];
    }
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    if constexpr (NW == 1) {
        int idx = 0, cnt = 20;
        const double v = ReduceScatter<20, 32>::run(acc, lane, idx, cnt);
        if ((lane & 1) == 0 && cnt > 0) mom[cell * 20 + idx] = v * (idx < 4 ? dV : G.m * dV);
    } else {
        block_sum_rs<20>(acc, red, fin_s);
        if (threadIdx.x < 20) mom[cell * 20 + threadIdx.x] = fin_s[threadIdx.x] * (threadIdx.x < 4 ? dV : G.m * dV);
    }
}

// One wave per cell (four cells per 256-thread block): lane l owns the v_x
// pencils at transverse positions t = l + 64 j (t = iy * N + iz), so the 20
// sums are reduced inside one wave, with no block barrier.
template <class T, int N>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8)))
moments3_cube_kernel(const T* __restrict__ f, double* __restrict__ mom, long long cells, VGrid G, XTable X) {
    constexpr int NT = (N * N + 63) / 64;
    const int lane = threadIdx.x & 63;
    const long long cell = (long long)xcd_work_index(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
    if (cell >= cells) return;
    const T* src = f + cell * (N * N * N);
    T fv[NT][N];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = lane + 64 * j;
#pragma unroll
        for (int k = 0; k < N; ++k) fv[j][k] = (t < N * N) ? ld_f<kRowsWholeLines<T, N>>(src + t + k * N * N) : T(0);
    }
    double acc[20];
#pragma unroll
    for (int q = 0; q < 20; ++q) acc[q] = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = lane + 64 * j;
        double S[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double g = (double)fv[j][k];
            S[0] += g;
            S[1] = fma(g, X.v[k], S[1]);
            S[2] = fma(g, X.v2[k], S[2]);
            S[3] = fma(g, X.v3[k], S[3]);
        }
        double a[20];
        pencil_moments(S, vc(G, 1, t / N), vc(G, 2, t % N), a);
#pragma unroll
        for (int q = 0; q < 20; ++q) acc[q] += a[q];
    }
    int idx = 0, cnt = 20;
    const double v = ReduceScatter<20, 32>::run(acc, lane, idx, cnt);
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    if ((lane & 1) == 0 && cnt > 0) mom[cell * 20 + idx] = v * (idx < 4 ? dV : G.m * dV);
}

// The same sums for FP32 blocks whose v_x planes are not whole cache lines
// (12^3: 576 B).  A cell is 6912 B, 54 whole lines: each wave reads its cell
// with 16-byte non-temporal loads (every wave instruction one 1 KB run of
// whole lines) into shared memory, then lane l takes its pencils from there
// as in moments3_cube_kernel (same arithmetic, same order).  The 27 KB of
// shared memory per workgroup allow five workgroups per CU, so the registers
// are capped for five waves per SIMD (96).  On the magnetotail grid: 869 ->
// 717 us per launch.
template <int N>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
moments3_staged_kernel(const float* __restrict__ f, double* __restrict__ mom, long long cells, VGrid G, XTable X) {
    typedef float F4 __attribute__((ext_vector_type(4)));
    constexpr int NV = N * N * N;
    constexpr int NT = (N * N + 63) / 64;
    constexpr int NQ = NV / 4;                    // 16-byte pieces of a cell
    static_assert(NV % 4 == 0 && (NV * 4) % 128 == 0, "cells of whole lines");
    __shared__ F4 buf[4][NQ];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long cell = (long long)xcd_work_index(blockIdx.x, gridDim.x) * 4 + w;
    if (cell >= cells) return;
    const F4* src = reinterpret_cast<const F4*>(f + cell * NV);
#pragma unroll
    for (int i = 0; i < (NQ + 63) / 64; ++i) {
        const int q = lane + 64 * i;
        if (q < NQ) buf[w][q] = __builtin_nontemporal_load(src + q);
    }
    // the wave reads back what its own lanes wrote: order its shared-memory
    // accesses (no other wave touches buf[w])
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const float* cb = reinterpret_cast<const float*>(buf[w]);
    double acc[20];
#pragma unroll
    for (int q = 0; q < 20; ++q) acc[q] = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = lane + 64 * j;
        double S[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double g = (double)((t < N * N) ? cb[t + k * N * N] : 0.0f);
            S[0] += g;
            S[1] = fma(g, X.v[k], S[1]);
            S[2] = fma(g, X.v2[k], S[2]);
            S[3] = fma(g, X.v3[k], S[3]);
        }
        double a[20];
        pencil_moments(S, vc(G, 1, t / N), vc(G, 2, t % N), a);
#pragma unroll
        for (int q = 0; q < 20; ++q) acc[q] += a[q];
    }
    int idx = 0, cnt = 20;
    const double v = ReduceScatter<20, 32>::run(acc, lane, idx, cnt);
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    if ((lane & 1) == 0 && cnt > 0) mom[cell * 20 + idx] = v * (idx < 4 ? dV : G.m * dV);
}

// Large cubic blocks (a cell's pencils do not fit one wave's registers): one
// block per cell; thread t sums the v_x pencils at transverse positions
// t, t + NTH, ... one pencil at a time, then a block reduction of the 20 sums.
// A 34^3 v_x plane is not a whole number of lines (4624 B in FP32), so the
// loads are ordinary and the caches merge the lines two wave accesses share
// (938 -> 839 us per 256x128x34^3 FP32 launch against non-temporal loads).
template <class T, int N, int NTH>
__global__ void __launch_bounds__(NTH)
moments3_big_kernel(const T* __restrict__ f, double* __restrict__ mom, VGrid G, XTable X) {
    __shared__ double red[(NTH / 64) * 20];
    __shared__ double fin_s[20];
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const T* src = f + cell * (N * N * N);
    double acc[20];
#pragma unroll
    for (int q = 0; q < 20; ++q) acc[q] = 0.0;
    for (int t = threadIdx.x; t < N * N; t += NTH) {
        T fv[N];
#pragma unroll
        for (int k = 0; k < N; ++k) fv[k] = ld_f<kRowsWholeLines<T, N>>(src + t + k * N * N);
        double Se[4] = {0.0, 0.0, 0.0, 0.0}, So[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double g = (double)fv[k];
            double* S = (k & 1) ? So : Se;
            S[0] += g;
            S[1] = fma(g, X.v[k], S[1]);
            S[2] = fma(g, X.v2[k], S[2]);
            S[3] = fma(g, X.v3[k], S[3]);
        }
        const double S[4] = {Se[0] + So[0], Se[1] + So[1], Se[2] + So[2], Se[3] + So[3]};
        double a[20];
        pencil_moments(S, vc(G, 1, t / N), vc(G, 2, t % N), a);
#pragma unroll
        for (int q = 0; q < 20; ++q) acc[q] += a[q];
    }
    block_sum_rs<20>(acc, red, fin_s);
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    if (threadIdx.x < 20) mom[cell * 20 + threadIdx.x] = fin_s[threadIdx.x] * (threadIdx.x < 4 ? dV : G.m * dV);
}

// Moment fitting of one cubic cell per block (see fit3_kernel for the steps).
// Per element: two exponentials of a quadratic in v_x whose other terms are
// per-thread constants, the exchange and clip, and FP64 pencil sums.
// exp(-q) with q scaled by log2(e) in FP32 (one v_exp_f32), exp() in FP64.
template <class T> struct ExpK;
template <> struct ExpK<float> {
    static constexpr double scale = 1.4426950408889634;   // log2(e)
    static __device__ __forceinline__ float e(float q) { return __builtin_amdgcn_exp2f(-q); }
};
template <> struct ExpK<double> {
    static constexpr double scale = 1.0;
    static __device__ __forceinline__ double e(double q) { return exp(-q); }
};

template <class T>
struct QuadX {       // (m/2) w^T T^-1 w = axx wx^2 + bt wx + ct for fixed (wy, wz), times ExpK::scale
    T axx, bt, ct, ux;
    // a: (m/2) ExpK::scale T^-1 as (xx, xy, xz, yy, yz, zz); u: mean velocity
    __device__ __forceinline__ void set(const double* a, const double* u, double vy, double vz) {
        const double wy = vy - u[1], wz = vz - u[2];
        axx = (T)a[0];
        bt = (T)(2.0 * (a[1] * wy + a[2] * wz));
        ct = (T)(a[3] * wy * wy + 2.0 * a[4] * wy * wz + a[5] * wz * wz);
        ux = (T)u[0];
    }
    __device__ __forceinline__ T g(T vx) const {
        const T wx = vx - ux;
        return ExpK<T>::e(fma(fma(axx, wx, bt), wx, ct));
    }
};

// Per-cell set-up of the fitting (one thread per cell), so that the f pass
// carries no FP64 divisions, square roots or branches on the moments: the
// exponent coefficients of the two Maxwellians, the density n_V, the skip
// decision; the fluid state is rescaled by n_V/n_F in place.
struct FitCell {
    double aV[6], uV[3], aF[6], uF[3];
    double nV, ok;
};
static_assert(sizeof(FitCell) == kFitCellDoubles * sizeof(double), "FitCell layout");

// blockIdx.y: species of the set (their outputs one after the other); a launch
// of its own is 5 us on a grid of any size up to 32768 cells, bound by its chain
// of divisions and square roots.
struct FitSet {
    const double* mom_pre[2];
    double* U[2];
    double m[2], kscale[2];
};

__global__ void __launch_bounds__(256)
fit3_params_kernel(FitSet S, long long cells, FitCell* __restrict__ out, unsigned long long* __restrict__ counters) {
    __shared__ int nskip;
    const int sp = blockIdx.y;
    const double* __restrict__ mom_pre = S.mom_pre[sp];
    double* __restrict__ U = S.U[sp];
    const double m = S.m[sp], kscale = S.kscale[sp];
    out += sp * cells;
    if (threadIdx.x == 0) nskip = 0;
    __syncthreads();
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < cells) {
        double mp[10], Uc[10];
#pragma unroll
        for (int k = 0; k < 10; ++k) { mp[k] = mom_pre[c * 20 + k]; Uc[k] = U[c * 10 + k]; }
        const double nV = mp[0], nF = Uc[0];
        double uV[3] = {0, 0, 0}, TV[6], uF[3] = {0, 0, 0}, TF[6], iV[6] = {0, 0, 0, 0, 0, 0}, iF[6] = {0, 0, 0, 0, 0, 0};
        bool ok = nV > 1e-12 && nF > 1e-12;
        if (ok) {
            u_and_T(mp + 1, nV, m, uV, TV);
            u_and_T(Uc + 1, nF, m, uF, TF);
            ok = spd_inverse(TV, iV) && spd_inverse(TF, iF);
        }
        FitCell r;
        const double h = 0.5 * m * kscale;
#pragma unroll
        for (int k = 0; k < 6; ++k) { r.aV[k] = h * iV[k]; r.aF[k] = h * iF[k]; }
#pragma unroll
        for (int k = 0; k < 3; ++k) { r.uV[k] = uV[k]; r.uF[k] = uF[k]; }
        r.nV = nV;
        r.ok = ok ? 1.0 : 0.0;
        out[c] = r;
        if (ok) {
            const double sc = nV / nF;
#pragma unroll
            for (int k = 0; k < 10; ++k) U[c * 10 + k] = Uc[k] * sc;
        } else {
            atomicAdd(&nskip, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && counters && nskip) atomicAdd(&counters[1], (unsigned long long)nskip);
}

// One block of NW waves per cell; thread t owns the v_x pencils at transverse
// positions t + 64 NW j (j < NT).  Two passes over f held in registers: the
// normalisation sums of the two Maxwellians (exponentials and pencil sums in
// the storage type, FP64 across pencils), then the exchange, clip (counted
// per wave with a ballot), FP64 post-fit moments and the FP64 rescale.  The
// block sums use the reduce-scatter (block_sum_rs).
// Launch shapes: 16^3 two waves of two pencils per thread, 12^3 one wave of
// three pencils per lane.
constexpr int kFit16Waves = 2, kFit16Pencils = 2;
constexpr int kFit12Waves = 1, kFit12Pencils = 3;
template <class T, int N, int NW, int NT>
__global__ void __launch_bounds__(64 * NW)
fit3_cube_kernel(const T* fin, T* fout, const FitCell* __restrict__ P, double* __restrict__ mom_post,
                 unsigned* __restrict__ clip_part, VGrid G, XTable X, typename Bits<T>::U* __restrict__ max_out) {
    constexpr int NTH = 64 * NW;
    // every thread owns NT whole pencils (no idle positions to mask)
    constexpr bool kFull = NT * NTH == N * N;
    // keeping the pass-1 exponentials in registers pays while they fit
    constexpr bool kKeep = NT * N <= 48;
    __shared__ double red[NW * 21];
    __shared__ double fin_s[21];
    const int tid = threadIdx.x;
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    const T* src = fin + cell * (N * N * N);
    T* dst = fout + cell * (N * N * N);
    T fv[NT][N];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = tid + NTH * j;
#pragma unroll
        for (int k = 0; k < N; ++k)
            fv[j][k] = (kFull || t < N * N) ? __builtin_nontemporal_load(src + t + k * N * N) : T(0);
    }
    // v_x in the storage type: held in registers for the small blocks,
    // converted at each use for the large ones (register pressure)
    constexpr bool kVx = N <= 16;
    T vxr[kVx ? N : 1];
#pragma unroll
    for (int k = 0; k < (kVx ? N : 1); ++k) vxr[k] = (T)X.v[k];
    auto vx = [&](int k) -> T { return kVx ? vxr[k] : (T)X.v[k]; };
    const FitCell& C = P[cell];
    const bool ok = C.ok != 0.0;
    const double nV = C.nV;
    unsigned nclip = 0;     // clipped elements of this wave (the same in every lane)
    if (ok) {
        QuadX<T> qv[NT], qf[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int t = tid + NTH * j;
            const double vy = vc(G, 1, t / N), vz = vc(G, 2, t % N);
            qv[j].set(C.aV, C.uV, vy, vz);
            qf[j].set(C.aF, C.uF, vy, vz);
        }
        // pencil sums of the samples in the storage type (four interleaved
        // chains; the samples carry that type's rounding already), added
        // across pencils in FP64
        double s[2] = {0.0, 0.0};
        T gv[kKeep ? NT : 1][kKeep ? N : 1], gf[kKeep ? NT : 1][kKeep ? N : 1];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (kFull || tid + NTH * j < N * N) {
                T pa[4] = {T(0), T(0), T(0), T(0)}, pb[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const T a = qv[j].g(vx(k)), b = qf[j].g(vx(k));
                    if constexpr (kKeep) {
                        gv[j][k] = a;
                        gf[j][k] = b;
                    }
                    pa[k & 3] += a;
                    pb[k & 3] += b;
                }
                s[0] += (double)((pa[0] + pa[1]) + (pa[2] + pa[3]));
                s[1] += (double)((pb[0] + pb[1]) + (pb[2] + pb[3]));
            }
        }
        block_sum_rs<2>(s, red, fin_s);
        const T A = (T)(nV / (fin_s[0] * dV));
        const T Bc = (T)(nV / (fin_s[1] * dV));
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const bool act = kFull || tid + NTH * j < N * N;
#pragma unroll
            for (int k = 0; k < N; ++k) {
                T x;
                if constexpr (kKeep) {
                    x = fv[j][k] - A * gv[j][k] + Bc * gf[j][k];
                } else {
                    x = fv[j][k] - A * qv[j].g(vx(k)) + Bc * qf[j].g(vx(k));
                }
                const bool neg = x < T(0);
                nclip += (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(act && neg));
                fv[j][k] = act ? (neg ? T(0) : x) : T(0);
            }
        }
    }
    // raw moments of the clipped f'' (FP64 pencil sums)
    double acc[21];
#pragma unroll
    for (int q = 0; q < 20; ++q) acc[q] = 0.0;
    acc[20] = (tid & (kWave - 1)) == 0 ? (double)nclip : 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = tid + NTH * j;
        // pencil sums over even and odd v_x separately (two independent chains)
        double Se[4] = {0.0, 0.0, 0.0, 0.0}, So[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double g = (double)fv[j][k];
            double* S = (k & 1) ? So : Se;
            S[0] += g;
            S[1] = fma(g, X.v[k], S[1]);
            S[2] = fma(g, X.v2[k], S[2]);
            S[3] = fma(g, X.v3[k], S[3]);
        }
        const double S[4] = {Se[0] + So[0], Se[1] + So[1], Se[2] + So[2], Se[3] + So[3]};
        double a[20];
        pencil_moments(S, vc(G, 1, t / N), vc(G, 2, t % N), a);
#pragma unroll
        for (int q = 0; q < 20; ++q) acc[q] += a[q];
    }
    block_sum_rs<21>(acc, red, fin_s);
    const double scale = ok ? nV / (fin_s[0] * dV) : 1.0;
    const T sc = (T)scale;     // 1 exactly when the cell is skipped
    T mx = T(0);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = tid + NTH * j;
        if (kFull || t < N * N) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const T o = fv[j][k] * sc;
                __builtin_nontemporal_store(o, dst + t + k * N * N);
                mx = fmax(mx, o);
            }
        }
    }
    if (mom_post && tid < 20) mom_post[cell * 20 + tid] = fin_s[tid] * (tid < 4 ? dV : G.m * dV) * scale;
    if (clip_part && tid == 0) clip_part[blockIdx.x] = (unsigned)fin_s[20];
    if (max_out) block_max_part(mx, max_out);
}

// Moment fitting of one large cubic cell per block (34^3) without holding the
// cell: the normalisation sums need only the two Maxwellians, so the block
// computes them first; f is then streamed once, pencil by pencil (thread t
// owns the v_x pencils t + NTH j), exchanged, clipped, summed into the FP64
// post-fit moments and stored unscaled, through the caches.  Where the
// density rescale factor rounds to one in the storage type the stored values
// are final, equal to fit3_cube_kernel's; elsewhere (a quarter to a third of
// the cells in FP32) each thread reads back the values it stored, which are
// mostly still in L2, and rescales them.  No 157 KB (FP32) or 314 KB (FP64)
// cell is held in registers or shared memory, so several cells share a CU.
// The loads are ordinary too: a 34^3 v_x plane is not a whole number of
// lines, and the caches merge the lines two wave accesses share (FP32: 2.82
// -> 2.47 ms per 256x128x34^3 launch; FP64 unchanged).
// The arithmetic is fit3_cube_kernel's (pencil sums of the samples in four
// chains in FP32, two in FP64; samples computed again in the exchange).
template <class T, int N, int NTH>
__global__ void __launch_bounds__(NTH)
fit3_stream_kernel(const T* fin, T* fout, const FitCell* __restrict__ P, double* __restrict__ mom_post,
                   unsigned* __restrict__ clip_part, VGrid G, XTable X, typename Bits<T>::U* __restrict__ max_out) {
    constexpr int NN = N * N;
    constexpr int NS = (NN + NTH - 1) / NTH;     // pencil sets
    constexpr int NW = NTH / kWave;
    constexpr int CH = sizeof(T) == 4 ? 4 : 2;   // pass-1 sum chains
    constexpr unsigned XB = NN * sizeof(T);      // bytes between v_x planes
    static_assert(NTH % kWave == 0, "launch shape");
    __shared__ double red[NW * 21];
    __shared__ double fin_s[21];
    const int tid = threadIdx.x;
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(fin + cell * (N * NN)), 0, N * XB, kBufWord3);
    const auto rd = __builtin_amdgcn_make_buffer_rsrc(fout + cell * (N * NN), 0, N * XB, kBufWord3);
    auto act = [&](int j) { return tid + NTH * j < NN; };
    const FitCell& C = P[cell];
    const bool ok = C.ok != 0.0;
    const double nV = C.nV;
    T A = T(0), Bc = T(0);
    if (ok) {
        // normalisation sums of the two Maxwellians (FP64 across pencils)
        double s[2] = {0.0, 0.0};
#pragma unroll 1
        for (int j = 0; j < NS; ++j) {
            if (act(j)) {
                const int t = tid + NTH * j;
                QuadX<T> qv, qf;
                qv.set(C.aV, C.uV, vc(G, 1, t / N), vc(G, 2, t % N));
                qf.set(C.aF, C.uF, vc(G, 1, t / N), vc(G, 2, t % N));
                T pa[CH], pb[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) pa[c] = pb[c] = T(0);
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    pa[k % CH] += qv.g((T)X.v[k]);
                    pb[k % CH] += qf.g((T)X.v[k]);
                }
                if constexpr (CH == 4) {
                    s[0] += (double)((pa[0] + pa[1]) + (pa[2] + pa[3]));
                    s[1] += (double)((pb[0] + pb[1]) + (pb[2] + pb[3]));
                } else {
                    s[0] += (double)(pa[0] + pa[1]);
                    s[1] += (double)(pb[0] + pb[1]);
                }
            }
        }
        block_sum_rs<2>(s, red, fin_s);
        A = (T)(nV / (fin_s[0] * dV));
        Bc = (T)(nV / (fin_s[1] * dV));
    }
    // exchange, clip, FP64 moments and the unscaled store, one pencil at a time
    double acc[21];
#pragma unroll
    for (int q = 0; q < 21; ++q) acc[q] = 0.0;
    unsigned nclip = 0;     // clipped elements of this wave (the same in every lane)
    T mx = T(0);
#pragma unroll 1
    for (int j = 0; j < NS; ++j) {
        const bool a = act(j);
        const int t = a ? tid + NTH * j : 0;
        const unsigned po = (unsigned)t * sizeof(T);
        T g[N];
#pragma unroll
        for (int k = 0; k < N; ++k) g[k] = a ? buf_ld<kBufCached>(rs, po, k * XB, T()) : T(0);
        if (ok) {
            QuadX<T> qv, qf;
            qv.set(C.aV, C.uV, vc(G, 1, t / N), vc(G, 2, t % N));
            qf.set(C.aF, C.uF, vc(G, 1, t / N), vc(G, 2, t % N));
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const T x = g[k] - A * qv.g((T)X.v[k]) + Bc * qf.g((T)X.v[k]);
                const bool neg = x < T(0);
                nclip += (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(a && neg));
                g[k] = neg ? T(0) : x;
            }
        }
        if (a) {
            double Se[4] = {0.0, 0.0, 0.0, 0.0}, So[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const double v = (double)g[k];
                double* S = (k & 1) ? So : Se;
                S[0] += v;
                S[1] = fma(v, X.v[k], S[1]);
                S[2] = fma(v, X.v2[k], S[2]);
                S[3] = fma(v, X.v3[k], S[3]);
                buf_st<kBufCached>(g[k], rd, po, k * XB);
                mx = fmax(mx, g[k]);
            }
            const double S[4] = {Se[0] + So[0], Se[1] + So[1], Se[2] + So[2], Se[3] + So[3]};
            double m[20];
            pencil_moments(S, vc(G, 1, t / N), vc(G, 2, t % N), m);
#pragma unroll
            for (int q = 0; q < 20; ++q) acc[q] += m[q];
        }
    }
    acc[20] = (tid & (kWave - 1)) == 0 ? (double)nclip : 0.0;
    block_sum_rs<21>(acc, red, fin_s);
    const double scale = ok ? nV / (fin_s[0] * dV) : 1.0;
    const T sc = (T)scale;     // 1 exactly when the cell is skipped
    if (sc != T(1)) {          // uniform over the block
        mx = T(0);
#pragma unroll 1
        for (int j = 0; j < NS; ++j) {
            if (act(j)) {
                const unsigned po = (unsigned)(tid + NTH * j) * sizeof(T);
                T g[N];
#pragma unroll
                for (int k = 0; k < N; ++k) g[k] = buf_ld<kBufCached>(rd, po, k * XB, T());
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const T o = g[k] * sc;
                    buf_st(o, rd, po, k * XB);
                    mx = fmax(mx, o);
                }
            }
        }
    }
    if (mom_post && tid < 20) mom_post[cell * 20 + tid] = fin_s[tid] * (tid < 4 ? dV : G.m * dV) * scale;
    if (clip_part && tid == 0) clip_part[blockIdx.x] = (unsigned)fin_s[20];
    if (max_out) block_max_part(mx, max_out);
}

// Moment fitting on any velocity grid with axes up to 32 (the general form of
// fit3_cube_kernel): one block per cell, thread t owns the v_x pencils t,
// t + blockDim, ...  A first pass over the grid sums the two Maxwellians (no
// memory traffic), a second reads f, exchanges, clips, sums the moments and
// leaves the result in shared memory, from where the same thread rescales and
// stores it.  Between the passes the kinetic samples wait in that memory, the
// fluid's are formed again.  exp(-q) with q summed in the order of Quad::g,
// added in FP64.
// 100 x 50 cells of 20x16x24 FP32: 283 us by the kernel that held 32 strided
// elements per thread with their indices formed by division and row sums
// through shared memory, now 99 (code for the exact pencil length, as in the
// moments: 119, too many registers).
template <class T>
struct Quad {       // (m/2) w^T T^-1 w for fixed (v_y, v_z)
    T axx, axz, azz, ux;
    T wz, xy, yy, wy;      // w_z, a_xy w_y, a_yy w_y + a_yz w_z, w_y
    __device__ __forceinline__ void set(const double* a, const double* u, T vy, T vz) {
#pragma clang fp contract(off)
        axx = (T)a[0];
        axz = (T)(2.0 * a[2]);
        ux = (T)u[0];
        wy = vy - (T)u[1];
        wz = vz - (T)u[2];
        xy = wy * (T)(2.0 * a[1]);
        yy = fma(wz, (T)(2.0 * a[4]), wy * (T)a[3]);
        azz = wz * (T)a[5];
    }
    __device__ __forceinline__ T g(T vx) const {
#pragma clang fp contract(off)
        const T wx = vx - ux;
        const T q = fma(wz, azz, fma(wy, yy, wx * fma(wz, axz, fma(wx, axx, xy))));
        return expo<T>(-q);
    }
};

template <class T>
__global__ void __launch_bounds__(256)
fit3_kernel(const T* fin, T* fout, const FitCell* __restrict__ P, double* __restrict__ mom_post,
            unsigned* __restrict__ clip_part, VGrid G, XTable X, typename Bits<T>::U* __restrict__ max_out) {
    extern __shared__ unsigned char smem_raw[];
    T* blk = reinterpret_cast<T*>(smem_raw);
    __shared__ double red[4 * 21];
    __shared__ double fin_s[21];
    const int tid = threadIdx.x, nthr = blockDim.x;
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const int npen = G.nvy * G.nvz, nvx = G.nvx;
    const double dV = G.dv[0] * G.dv[1] * G.dv[2];
    const T* src = fin + cell * npen * nvx;
    T* dst = fout + cell * npen * nvx;
    const FitCell& C = P[cell];
    const bool ok = C.ok != 0.0;
    const double nV = C.nV;
    T A = T(0), Bc = T(0);
    auto at = [&](int t, Quad<T>& qv, Quad<T>& qf) {
        const int iy = row_of(t, G.inv_nvz);
        const T vy = (T)vc(G, 1, iy), vz = (T)vc(G, 2, t - iy * G.nvz);
        qv.set(C.aV, C.uV, vy, vz);
        qf.set(C.aF, C.uF, vy, vz);
    };
    if (ok) {
        double s[2] = {0.0, 0.0};
        for (int t = tid; t < npen; t += nthr) {
            Quad<T> qv, qf;
            at(t, qv, qf);
            double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
            for (int k = 0; k < nvx; ++k) {
                const T gv = qv.g((T)X.v[k]);
                blk[k * npen + t] = gv;
                s0 += (double)gv;
                s1 += (double)qf.g((T)X.v[k]);
            }
            s[0] += s0;
            s[1] += s1;
        }
        block_sum_rs<2>(s, red, fin_s);
        A = (T)(nV / (fin_s[0] * dV));
        Bc = (T)(nV / (fin_s[1] * dV));
    }
    double acc[21];
#pragma unroll
    for (int q = 0; q < 21; ++q) acc[q] = 0.0;
    unsigned nclip = 0;
    for (int t = tid; t < npen; t += nthr) {
        Quad<T> qv, qf;
        if (ok) at(t, qv, qf);
        double S[4] = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = 0; k0 < nvx; k0 += 8) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = k0 + u < nvx ? src[(unsigned)((k0 + u) * npen + t)] : T(0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (k0 + u >= nvx) break;
                const int k = k0 + u;
                T x = v[u];
                if (ok) {
                    x = fma(Bc, qf.g((T)X.v[k]), fma(-A, blk[k * npen + t], x));
                    nclip += x < T(0) ? 1u : 0u;
                    x = fmax(x, T(0));
                }
                blk[k * npen + t] = x;
                const double g = (double)x;
                S[0] += g;
                S[1] = fma(g, X.v[k], S[1]);
                S[2] = fma(g, X.v2[k], S[2]);
                S[3] = fma(g, X.v3[k], S[3]);
            }
        }
        const int iy = row_of(t, G.inv_nvz);
        double a[20];
        pencil_moments(S, vc(G, 1, iy), vc(G, 2, t - iy * G.nvz), a);
#pragma unroll
        for (int q = 0; q < 20; ++q) acc[q] += a[q];
    }
    acc[20] = (double)nclip;
    block_sum_rs<21>(acc, red, fin_s);
    const double scale = ok ? nV / (fin_s[0] * dV) : 1.0;
    const T sc = (T)scale;     // 1 exactly when the cell is skipped
    T mx = T(0);
    for (int t = tid; t < npen; t += nthr) {
#pragma unroll 8
        for (int k = 0; k < nvx; ++k) {
            const T o = ok ? blk[k * npen + t] * sc : blk[k * npen + t];
            dst[(unsigned)(k * npen + t)] = o;
            mx = fmax(mx, o);
        }
    }
    if (mom_post && tid < 20) mom_post[cell * 20 + tid] = fin_s[tid] * (tid < 4 ? dV : G.m * dV) * scale;
    if (clip_part && tid == 0) clip_part[cell] = (unsigned)fin_s[20];
    if (max_out) block_max_part(mx, max_out);
}

template <class T>
__global__ void __launch_bounds__(256)
fit1_kernel(const T* fin, T* fout, const double* __restrict__ mom_pre, const double* Uin, double* U,
            double* __restrict__ mom_post, unsigned long long* __restrict__ counters, int nv, double vlo,
            double dv, double mass, typename Bits<T>::U* __restrict__ max_out) {
    extern __shared__ unsigned char smem_raw[];
    T* g = reinterpret_cast<T*>(smem_raw);
    __shared__ double red[5 * 4];
    const long long cell = blockIdx.x;
    const T* src = fin + cell * nv;
    T* dst = fout + cell * nv;
    const double nV = mom_pre[cell * 4 + 0];
    const double Un = Uin[cell * 3 + 0], Unu = Uin[cell * 3 + 1], UP = Uin[cell * 3 + 2];
    bool ok = nV > 1e-12 && Un > 1e-12;
    double uV = 0, TV = 0, uF = 0, TF = 0;
    if (ok) {
        uV = mom_pre[cell * 4 + 1] / nV;
        TV = (mom_pre[cell * 4 + 2] - mass * nV * uV * uV) / nV;
        uF = Unu / Un;
        TF = (UP - mass * Un * uF * uF) / Un;
        ok = TV > 0.0 && TF > 0.0;
    }
    const T aV = (T)(0.5 * mass / TV), aF = (T)(0.5 * mass / TF);
    double s[2] = {0.0, 0.0};
    if (ok) {
        for (int j = threadIdx.x; j < nv; j += blockDim.x) {
            const double v = vlo + (j + 0.5) * dv;
            const T wv = (T)(v - uV), wf = (T)(v - uF);
            s[0] += (double)expo<T>(-aV * wv * wv);
            s[1] += (double)expo<T>(-aF * wf * wf);
        }
    }
    block_sum<2>(s, red);
    const T A = ok ? (T)(nV / (s[0] * dv)) : T(0);
    const T Bc = ok ? (T)(nV / (s[1] * dv)) : T(0);
    double acc[5] = {0, 0, 0, 0, 0};
    for (int j = threadIdx.x; j < nv; j += blockDim.x) {
        T x = src[j];
        if (ok) {
            const double v = vlo + (j + 0.5) * dv;
            const T wv = (T)(v - uV), wf = (T)(v - uF);
            x = x - A * expo<T>(-aV * wv * wv) + Bc * expo<T>(-aF * wf * wf);
            if (x < T(0)) acc[4] += 1.0;
            x = fmax(x, T(0));
        }
        g[j] = x;
        const double v = vlo + (j + 0.5) * dv;
        const double xd = (double)x, xv = xd * v;
        acc[0] += xd;
        acc[1] += xv;
        acc[2] += xv * v;
        acc[3] += xv * v * v;
    }
    block_sum<5>(acc, red);
    const double scale = ok ? nV / (acc[0] * dv) : 1.0;
    const T sc = (T)scale;
    T mx = T(0);
    for (int j = threadIdx.x; j < nv; j += blockDim.x) {
        const T o = ok ? g[j] * sc : g[j];
        dst[j] = o;
        mx = fmax(mx, o);
    }
    if (threadIdx.x == 0) {
        if (mom_post) {
            mom_post[cell * 4 + 0] = acc[0] * dv * scale;
            mom_post[cell * 4 + 1] = acc[1] * dv * scale;
            mom_post[cell * 4 + 2] = mass * acc[2] * dv * scale;
            mom_post[cell * 4 + 3] = mass * acc[3] * dv * scale;
        }
        if (ok || Uin != U) {
            const double r = ok ? nV / Un : 1.0;
            U[cell * 3 + 0] = Un * r;
            U[cell * 3 + 1] = Unu * r;
            U[cell * 3 + 2] = UP * r;
        }
        if (counters) {
            if (acc[4] > 0) atomicAdd(&counters[0], (unsigned long long)acc[4]);
            if (!ok) atomicAdd(&counters[1], 1ull);
        }
    }
    if (max_out) block_max_part(mx, max_out);
}

// ------------------------------------------------------------ launchers ----
static int threads_for(int work) {
    int t = ((work + 63) / 64) * 64;
    return t > 256 ? 256 : (t < 64 ? 64 : t);
}

static XTable xtable(const VGridArgs& a) {
    XTable X{};
    for (int k = 0; k < a.nv[0] && k < kBigCube; ++k) {
        const double v = a.lo[0] + (k + 0.5) * a.dv[0];
        X.v[k] = v;
        X.v2[k] = v * v;
        X.v3[k] = v * v * v;
    }
    return X;
}

static int cube_edge(const VGridArgs& a) {
    const bool cube = a.nv[0] == a.nv[1] && a.nv[1] == a.nv[2];
    return (cube && (a.nv[0] == 8 || a.nv[0] == 12 || a.nv[0] == 16 || a.nv[0] == kBigCube)) ? a.nv[0] : 0;
}

template <class T>
hipError_t launch_moments3(const T* f, double* mom, long long cells, const VGridArgs& a, hipStream_t st) {
    VGrid G{a.nv[0], a.nv[1], a.nv[2], {a.lo[0], a.lo[1], a.lo[2]}, {a.dv[0], a.dv[1], a.dv[2]}, a.m, 1.0f / (float)a.nv[2]};
    const int N = cube_edge(a);
    if (N) {
        const XTable X = xtable(a);
        const dim3 grid((unsigned)((cells + 3) / 4)), blk(256);
        if (N == 16) hipLaunchKernelGGL((moments3_cube_kernel<T, 16>), grid, blk, 0, st, f, mom, cells, G, X);
        if (N == 12) {
            // 16-byte pieces need a 16-byte aligned f (any allocation is)
            if constexpr (sizeof(T) == 4) {
                if (reinterpret_cast<uintptr_t>(f) % 16 == 0)
                    hipLaunchKernelGGL((moments3_staged_kernel<12>), grid, blk, 0, st, f, mom, cells, G, X);
                else
                    hipLaunchKernelGGL((moments3_cube_kernel<T, 12>), grid, blk, 0, st, f, mom, cells, G, X);
            } else {
                hipLaunchKernelGGL((moments3_cube_kernel<T, 12>), grid, blk, 0, st, f, mom, cells, G, X);
            }
        }
        if (N == 8) hipLaunchKernelGGL((moments3_cube_kernel<T, 8>), grid, blk, 0, st, f, mom, cells, G, X);
        if (N == kBigCube)
            hipLaunchKernelGGL((moments3_big_kernel<T, kBigCube, 256>), dim3((unsigned)cells), blk, 0, st, f, mom,
                               G, X);
        return hipGetLastError();
    }
    const XTable X = xtable(a);
    // One wave per cell where that fills the chip (its reduction is a quarter of
    // the work of four waves' and needs no barrier: 20000 cells of 10^3 34 us
    // per call against 57) or where a wave has at most two pencils per lane; four waves
    // for few large cells (1000 of 20x16x24: 9.8 us against 18.1).
    if (a.nv[1] * a.nv[2] <= 128 || cells >= 4096)
        hipLaunchKernelGGL((moments3_kernel<T, 1>), dim3((unsigned)((cells + 3) / 4)), dim3(256), 0, st, f, mom, cells,
                           G, X);
    else
        hipLaunchKernelGGL((moments3_kernel<T, 4>), dim3((unsigned)cells), dim3(256), 0, st, f, mom, cells, G, X);
    return hipGetLastError();
}

template <class T>
hipError_t launch_moments1(const T* f, double* mom, long long cells, int nv, double vlo, double dv, double m,
                           hipStream_t st) {
    hipLaunchKernelGGL((moments1_kernel<T>), dim3((unsigned)cells), dim3(threads_for(nv)), 0, st, f, mom, nv, vlo, dv,
                       m);
    return hipGetLastError();
}

// The maxima and clip counts of the fits of a step (up to two species) from
// their per-block partials, all in one launch: block (or block row) 2 s folds
// species s's maxima into its slot, 2 s + 1 adds its clip counts to
// counters[0].  Up to kFoldOne partials each: one 1024-thread block per fold
// (at 32768 cells 4.6 us for both species, where two launches per fold took
// 8 x 3-10 us); more: ranges into a stage of 64-bit entries right behind the
// partials, then one wave per fold.  Counts are integers and the only
// unordered additions are two atomic ones: exact in any order.
template <class U>
struct FitFold {
    const U* part[VL_MAX_SPECIES];
    U* slot[VL_MAX_SPECIES];                  // null: no maximum to fold
    const unsigned* clips[VL_MAX_SPECIES];
    unsigned long long* counters;             // null: no counts wanted
    long long n;
};

__device__ __forceinline__ unsigned long long wave_count(unsigned long long acc) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kWave);
    return acc;
}

template <class U>
__global__ void __launch_bounds__(1024) fit_fold_kernel(FitFold<U> F) {
    const int s = blockIdx.x >> 1, n = (int)F.n;
    if ((blockIdx.x & 1) == 0) {
        if (F.slot[s]) fold_max_block<U>(F.part[s], n, F.slot[s]);
        return;
    }
    if (!F.counters) return;
    __shared__ unsigned long long red[1024 / kWave];
    const unsigned* clips = F.clips[s];
    const int tid = threadIdx.x;
    typedef unsigned Vec __attribute__((ext_vector_type(4)));
    const int nvec = ((uintptr_t)clips & 15u) ? 0 : n / 4;
    unsigned long long acc = 0;
#pragma unroll 8
    for (int i = tid; i < nvec; i += 1024) {
        const Vec v = reinterpret_cast<const Vec*>(clips)[i];
        acc += (unsigned long long)v[0] + v[1] + v[2] + v[3];
    }
    for (int i = nvec * 4 + tid; i < n; i += 1024) acc += clips[i];
    acc = wave_count(acc);
    if ((tid & (kWave - 1)) == 0) red[tid / kWave] = acc;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 1024 / kWave; ++w) acc += red[w];
        if (acc) atomicAdd(F.counters, acc);
    }
}

// First level for long partials: block x of row y folds its range into entry x
// of the row's stage.
template <class U>
__global__ void __launch_bounds__(256) fit_stage_kernel(FitFold<U> F, long long chunk) {
    const int s = blockIdx.y >> 1;
    const bool count = (blockIdx.y & 1) != 0;
    if (count ? !F.counters : !F.slot[s]) return;
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = lo + chunk < F.n ? lo + chunk : F.n;
    __shared__ unsigned long long red[256 / kWave];
    unsigned long long acc = 0;
    for (long long b = lo; b < hi; b += 8 * 256) {
        unsigned long long v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long long i = b + u * 256 + threadIdx.x;
            v[u] = i < hi ? (count ? (unsigned long long)F.clips[s][i] : (unsigned long long)F.part[s][i]) : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = count ? acc + v[u] : (v[u] > acc ? v[u] : acc);
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const unsigned long long y = __shfl_xor(acc, o, kWave);
        acc = count ? acc + y : (y > acc ? y : acc);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / kWave; ++w) acc = count ? acc + red[w] : (red[w] > acc ? red[w] : acc);
        const void* part = count ? (const void*)F.clips[s] : (const void*)F.part[s];
        auto* stage = (unsigned long long*)((char*)part + fin_stage(F.n, count ? sizeof(unsigned) : sizeof(U)));
        stage[blockIdx.x] = acc;
    }
}

template <class U>
__global__ void __launch_bounds__(kWave) fit_final_kernel(FitFold<U> F, int g) {
    const int s = blockIdx.x >> 1;
    const bool count = (blockIdx.x & 1) != 0;
    if (count ? !F.counters : !F.slot[s]) return;
    const void* part = count ? (const void*)F.clips[s] : (const void*)F.part[s];
    const auto* stage = (const unsigned long long*)((const char*)part +
                                                    fin_stage(F.n, count ? sizeof(unsigned) : sizeof(U)));
    unsigned long long acc = (int)threadIdx.x < g ? stage[threadIdx.x] : 0ull;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const unsigned long long y = __shfl_xor(acc, o, kWave);
        acc = count ? acc + y : (y > acc ? y : acc);
    }
    if (threadIdx.x != 0) return;
    if (!count) *F.slot[s] = (U)acc;
    else if (acc) atomicAdd(F.counters, acc);
}

template <class T>
hipError_t launch_fit_fold(int ns, const MaxSink* sinks, unsigned* const* clips, void* counters, long long cells,
                           hipStream_t st) {
    using U = typename Bits<T>::U;
    FitFold<U> F{};
    F.counters = (unsigned long long*)counters;
    F.n = cells;
    bool any = counters != nullptr;
    for (int s = 0; s < ns; ++s) {
        const bool fold = sinks[s].slot && !sinks[s].direct(cells);
        F.part[s] = (const U*)sinks[s].part;
        F.slot[s] = fold ? (U*)sinks[s].slot : nullptr;
        F.clips[s] = clips[s];
        any = any || fold;
    }
    if (!any) return hipSuccess;
    if (cells <= kFoldOne) {
        hipLaunchKernelGGL((fit_fold_kernel<U>), dim3(2 * ns), dim3(1024), 0, st, F);
        return hipGetLastError();
    }
    const FinSplit fs = fin_split(cells);
    hipLaunchKernelGGL((fit_stage_kernel<U>), dim3(fs.blocks, 2 * ns), dim3(256), 0, st, F, fs.chunk);
    hipLaunchKernelGGL((fit_final_kernel<U>), dim3(2 * ns), dim3(kWave), 0, st, F, fs.blocks);
    return hipGetLastError();
}

template <class T>
hipError_t launch_fit3_params(int ns, const double* const* mom_pre, double* const* U, const VGridArgs* a,
                              long long cells, double* params, void* counters, hipStream_t st) {
    if (ns < 1 || ns > 2) return hipErrorInvalidValue;
    FitSet S{};
    for (int k = 0; k < ns; ++k) {
        S.mom_pre[k] = mom_pre[k];
        S.U[k] = U[k];
        S.m[k] = a[k].m;
        S.kscale[k] = cube_edge(a[k]) ? ExpK<T>::scale : 1.0;
    }
    hipLaunchKernelGGL(fit3_params_kernel, dim3((unsigned)((cells + 255) / 256), ns), dim3(256), 0, st, S, cells,
                       reinterpret_cast<FitCell*>(params), (unsigned long long*)counters);
    return hipGetLastError();
}

template <class T>
hipError_t launch_fit3(const T* fin, T* fout, double* mom_post, void* counters, long long cells, const VGridArgs& a,
                       const MaxSink& sink, unsigned* clip_part, const double* params, hipStream_t st) {
    VGrid G{a.nv[0], a.nv[1], a.nv[2], {a.lo[0], a.lo[1], a.lo[2]}, {a.dv[0], a.dv[1], a.dv[2]}, a.m, 1.0f / (float)a.nv[2]};
    auto* mo = sink.target<T>(cells);
    unsigned* cp = counters ? clip_part : nullptr;
    const int N = cube_edge(a);
    const XTable X = xtable(a);
    const dim3 grid((unsigned)cells);
    const FitCell* P = reinterpret_cast<const FitCell*>(params);
    if (N) {
        // waves per cell and pencils per thread: every lane busy for 16^3, 3/4 for 12^3
        if constexpr (sizeof(T) == 4) {
            if (N == 16) hipLaunchKernelGGL((fit3_cube_kernel<T, 16, kFit16Waves, kFit16Pencils>), grid, dim3(64 * kFit16Waves), 0, st, fin, fout, P, mom_post, cp, G, X, mo);
            if (N == 12) hipLaunchKernelGGL((fit3_cube_kernel<T, 12, kFit12Waves, kFit12Pencils>), grid, dim3(64 * kFit12Waves), 0, st, fin, fout, P, mom_post, cp, G, X, mo);
            if (N == 8) hipLaunchKernelGGL((fit3_cube_kernel<T, 8, 1, 1>), grid, dim3(64), 0, st, fin, fout, P, mom_post, cp, G, X, mo);
            if (N == kBigCube)   // streamed: the cell is not held
                hipLaunchKernelGGL((fit3_stream_kernel<T, kBigCube, 256>), grid, dim3(256), 0, st, fin, fout, P,
                                   mom_post, cp, G, X, mo);
        } else {
            if (N == 16) hipLaunchKernelGGL((fit3_cube_kernel<T, 16, 4, 1>), grid, dim3(256), 0, st, fin, fout, P, mom_post, cp, G, X, mo);
            if (N == 12) hipLaunchKernelGGL((fit3_cube_kernel<T, 12, 3, 1>), grid, dim3(192), 0, st, fin, fout, P, mom_post, cp, G, X, mo);
            if (N == 8) hipLaunchKernelGGL((fit3_cube_kernel<T, 8, 1, 1>), grid, dim3(64), 0, st, fin, fout, P, mom_post, cp, G, X, mo);
            if (N == kBigCube)   // streamed: the cell is not held
                hipLaunchKernelGGL((fit3_stream_kernel<T, kBigCube, 256>), grid, dim3(256), 0, st, fin, fout, P,
                                   mom_post, cp, G, X, mo);
        }
        return hipGetLastError();
    }
    const int npen = a.nv[1] * a.nv[2];
    const size_t shm = sizeof(T) * (size_t)a.nv[0] * npen;
    int threads = pencil_threads(&npen, 1, shm, sizeof(T) == 4 ? 20 : 16, cells, false);
    if (threads > 256) threads = 256;
    hipLaunchKernelGGL((fit3_kernel<T>), grid, dim3(threads), shm, st, fin, fout, P, mom_post, cp, G, X, mo);
    return hipGetLastError();
}

template <class T>
hipError_t launch_fit1(const T* fin, T* fout, const double* mom_pre, const double* Uin, double* U, double* mom_post, void* counters,
                       long long cells, int nv, double vlo, double dv, double m, const MaxSink& sink,
                       hipStream_t st) {
    hipLaunchKernelGGL((fit1_kernel<T>), dim3((unsigned)cells), dim3(threads_for(nv)), sizeof(T) * (size_t)nv, st,
                       fin, fout, mom_pre, Uin, U, mom_post, (unsigned long long*)counters, nv, vlo, dv, m,
                       sink.target<T>(cells));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !sink.slot || sink.direct(cells)) return e;
    return launch_max_finalize<T>(sink.part, cells, sink.slot, st);
}

#define VL_INST(T)                                                                                              \
    template hipError_t launch_moments3<T>(const T*, double*, long long, const VGridArgs&, hipStream_t);         \
    template hipError_t launch_moments1<T>(const T*, double*, long long, int, double, double, double,            \
                                           hipStream_t);                                                        \
    template hipError_t launch_fit3_params<T>(int, const double* const*, double* const*, const VGridArgs*,    \
                                              long long, double*, void*, hipStream_t);                         \
    template hipError_t launch_fit3<T>(const T*, T*, double*, void*, long long, const VGridArgs&, const MaxSink&, \
                                       unsigned*, const double*, hipStream_t);      \
    template hipError_t launch_fit_fold<T>(int, const MaxSink*, unsigned* const*, void*, long long,             \
                                           hipStream_t);                                                       \
    template hipError_t launch_fit1<T>(const T*, T*, const double*, const double*, double*, double*, void*,     \
                                       long long, int, double, double, double, const MaxSink&, hipStream_t);
VL_INST(float)
VL_INST(double)
#undef VL_INST

}  // namespace vl

namespace vl {

// ------------------------------------------------------------ diagnostics --
// Deterministic two-level sums: block partials in a fixed order, then one
// block adds the partials in index order.
template <class T>
__global__ void __launch_bounds__(256)
partial_sum_kernel(const T* __restrict__ f, long long n, double* __restrict__ part) {
    __shared__ double red[4];
    double acc[1] = {0.0};
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        acc[0] += (double)f[i];
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) part[blockIdx.x] = acc[0];
}

__global__ void __launch_bounds__(256)
energy_partial_kernel(const double* __restrict__ mom, long long cells, int kmom, int dimv, double* __restrict__ part) {
    __shared__ double red[4];
    double acc[1] = {0.0};
    for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < cells; c += (long long)gridDim.x * blockDim.x)
        acc[0] += dimv == 3 ? 0.5 * (mom[c * kmom + 4] + mom[c * kmom + 7] + mom[c * kmom + 9]) : 0.5 * mom[c * kmom + 2];
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) part[blockIdx.x] = acc[0];
}

__global__ void __launch_bounds__(256)
finish_sum_kernel(const double* __restrict__ part, int np, double scale, double* __restrict__ out) {
    __shared__ double red[4];
    // thread t adds partials t, t+256, ... in order; then a fixed-order block sum
    double acc[1] = {0.0};
    for (int i = threadIdx.x; i < np; i += blockDim.x) acc[0] += part[i];
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) *out = acc[0] * scale;
}

template <class T>
hipError_t launch_mass_energy(const T* f, const double* mom, long long cells, long long nv, int kmom, int dimv,
                              double dV, double dX, double* out, double* part, hipStream_t st) {
    // out[0] = mass, out[1] = energy; part: 1024 doubles of scratch
    const int np = 1024;
    hipLaunchKernelGGL((partial_sum_kernel<T>), dim3(np), dim3(256), 0, st, f, cells * nv, part);
    hipLaunchKernelGGL(finish_sum_kernel, dim3(1), dim3(256), 0, st, part, np, dV * dX, out);
    hipLaunchKernelGGL(energy_partial_kernel, dim3(np), dim3(256), 0, st, mom, cells, kmom, dimv, part);
    hipLaunchKernelGGL(finish_sum_kernel, dim3(1), dim3(256), 0, st, part, np, dX, out + 1);
    return hipGetLastError();
}

template hipError_t launch_mass_energy<float>(const float*, const double*, long long, long long, int, int, double,
                                              double, double*, double*, hipStream_t);
template hipError_t launch_mass_energy<double>(const double*, const double*, long long, long long, int, int, double,
                                               double, double*, double*, hipStream_t);

}  // namespace vl
