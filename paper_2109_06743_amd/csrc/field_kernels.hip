// Field solvers for gfx950, all FP64 (the field update is kept in double
// precision because the energy exchange with the particles depends on it).
//
// 1X1V (Sec. 3.1): Gauss's law dE/dx = rho with eps0 = 1 and a uniform static
// ion background, solved with a discrete Fourier transform,
// E_i = (2/N) sum_{m=1}^{N/2-1} Im(rho_hat_m e^{i th}) / k_m, the mean and
// Nyquist modes dropped.  Written out that is a convolution of the density
// with g[n] = (2/N) sum_m sin(2 pi m n / N) / k_m, which depends on the grid
// only: g is tabulated once per context and a solve is N multiply-adds per
// cell, done by the kernels that need E.
//
// 2X3V (Sec. 2.1, Maxwell's equations, FDTD): Yee grid, mu0 = 1, eps0 = 1/c^2,
// x periodic, conducting walls in y with the tangential E (Ex, Ez) and normal
// B (By) odd about each wall.  A half step of length h = dt/2 is
//   B -= (h/2) curl E;  E += h c^2 (curl B - j);  B -= (h/2) curl E.
#include "vl_internal.h"

namespace vl {

// --------------------------------------------------------------- Poisson ---
// Table of the Green's function, one wave per entry 0 .. N/2 (g is odd).
__global__ void __launch_bounds__(256) poisson_green_kernel(int N, double L, double* __restrict__ g) {
    const int n = (int)blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (n > N / 2) return;
    double acc = 0.0;
    for (int m = 1 + lane; m < (N + 1) / 2; m += 64)
        acc += sinpi(2.0 * (double)(((long long)m * n) % N) / N) / (2.0 * M_PI * m / L);
    acc = 2.0 * wave_sum(acc) / N;
    if (2 * n == N || n == 0) acc = 0.0;
    if (lane == 0) {
        g[n] = acc;
        if (n > 0) g[N - n] = 2 * n == N ? 0.0 : -acc;
    }
}

// E at the centres from species moments [N][4].  Serial sums of FP64 sine and
// cosine calls, one thread per mode and then per cell, took 126 us at N = 256
// and 30 us at N = 64; this takes 5.
__global__ void __launch_bounds__(256)
poisson_kernel(const double* __restrict__ mom, int N, double q, const double* __restrict__ g, double* __restrict__ E) {
    __shared__ PoissonLds<1> L;
    const double* const src[1] = {mom};
    poisson_tile<1>(src, N, g, blockIdx.x * 64, q, L);
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x < 64 && i < N) E[i] = L.e[0][threadIdx.x];
}

hipError_t launch_poisson_green(int N, double L, double* g, hipStream_t st) {
    hipLaunchKernelGGL(poisson_green_kernel, dim3((N / 2 + 4) / 4), dim3(256), 0, st, N, L, g);
    return hipGetLastError();
}

hipError_t launch_poisson(const double* mom, int N, double q, const double* g, double* E, hipStream_t st) {
    hipLaunchKernelGGL(poisson_kernel, dim3((N + 63) / 64), dim3(256), 0, st, mom, N, q, g, E);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Yee ----
struct YeeView {
    double *Ex, *Ey, *Ez, *Bx, *By, *Bz;
    int nx, ny;
    int per;    // 1: periodic y (rows 0 and ny of the [ny+1] arrays are the same points)
};

__host__ __device__ inline YeeView yee_view(double* base, int nx, int ny) {
    const long long a = (long long)nx * ny, b = (long long)nx * (ny + 1);
    YeeView v;
    v.Ex = base;
    v.Ey = v.Ex + a;
    v.Ez = v.Ey + b;
    v.Bx = v.Ez + a;
    v.By = v.Bx + b;
    v.Bz = v.By + a;
    v.nx = nx;
    v.ny = ny;
    v.per = 0;
    return v;
}

// integer-row component (Ex, Ez) at row j: odd ghosts beyond conducting
// walls, wrapped rows when y is periodic
__device__ __forceinline__ double odd_row(const double* a, int j, int i, int nx, int ny, int per) {
    if (per) {
        if (j < 0) j += ny;
        if (j >= ny) j -= ny;
        return a[(long long)j * nx + i];
    }
    if (j < 0) return -a[(long long)(-1 - j) * nx + i];
    if (j >= ny) return -a[(long long)(2 * ny - 1 - j) * nx + i];
    return a[(long long)j * nx + i];
}

// B -= coef * curl E.  One thread per (jh in 0..ny, i).
__global__ void yee_curl_e_kernel(YeeView F, double coef, double dx, double dy) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int jh = blockIdx.y;
    const int nx = F.nx, ny = F.ny;
    if (i >= nx) return;
    const int ip = (i + 1 == nx) ? 0 : i + 1;
    const long long h = (long long)jh * nx;
    // Bx at (i, jh-1/2): (curl E)_x = dEz/dy
    const double dEz = (odd_row(F.Ez, jh, i, nx, ny, F.per) - odd_row(F.Ez, jh - 1, i, nx, ny, F.per)) / dy;
    F.Bx[h + i] -= coef * dEz;
    // Bz at (i+1/2, jh-1/2): (curl E)_z = dEy/dx - dEx/dy
    const double dEy = (F.Ey[h + ip] - F.Ey[h + i]) / dx;
    const double dEx = (odd_row(F.Ex, jh, i, nx, ny, F.per) - odd_row(F.Ex, jh - 1, i, nx, ny, F.per)) / dy;
    F.Bz[h + i] -= coef * (dEy - dEx);
    // By at (i+1/2, j): (curl E)_y = -dEz/dx
    if (jh < ny) F.By[h + i] += coef * (F.Ez[h + ip] - F.Ez[h + i]) / dx;
}

// E += coef c^2 (curl B - j); j = sum_s q_s M1_s at cell centres averaged to
// the E positions (j_y on a wall face is 0; periodic y: the mean across the
// seam).
struct Currents {
    const double* mom[2];   // per species: n u_x, n u_y, n u_z at offsets 1..3 of each cell's record
    double q[2];
    int ns;
    int stride;             // doubles per cell record (20: raw moments, 10: fluid state)
};

__device__ __forceinline__ double jc(const Currents& J, long long cell, int d) {
    double s = 0.0;
    for (int k = 0; k < J.ns; ++k) s += J.q[k] * J.mom[k][cell * J.stride + 1 + d];
    return s;
}

__global__ void yee_curl_b_kernel(YeeView F, Currents J, double coef, double c2, double dx, double dy) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int jh = blockIdx.y;
    const int nx = F.nx, ny = F.ny;
    if (i >= nx) return;
    const int im = (i == 0) ? nx - 1 : i - 1;
    const int ip = (i + 1 == nx) ? 0 : i + 1;
    const long long h = (long long)jh * nx;
    // Ey at (i, jh-1/2): (curl B)_y = -dBz/dx
    double jy = 0.0;
    if (jh > 0 && jh < ny) jy = 0.5 * (jc(J, h - nx + i, 1) + jc(J, h + i, 1));
    else if (F.per) jy = 0.5 * (jc(J, (long long)(ny - 1) * nx + i, 1) + jc(J, i, 1));   // across the seam
    F.Ey[h + i] += coef * c2 * (-(F.Bz[h + i] - F.Bz[h + im]) / dx - jy);
    if (jh < ny) {
        // Ex at (i+1/2, j): (curl B)_x = dBz/dy
        const double jx = 0.5 * (jc(J, h + i, 0) + jc(J, h + ip, 0));
        F.Ex[h + i] += coef * c2 * ((F.Bz[h + nx + i] - F.Bz[h + i]) / dy - jx);
        // Ez at (i, j): (curl B)_z = dBy/dx - dBx/dy
        const double jz = jc(J, h + i, 2);
        F.Ez[h + i] += coef * c2 * ((F.By[h + i] - F.By[h + im]) / dx - (F.Bx[h + nx + i] - F.Bx[h + i]) / dy - jz);
    }
}

__global__ void cell_fields_kernel(YeeView F, double* __restrict__ E, double* __restrict__ B) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    const int nx = F.nx;
    if (i >= nx) return;
    const int im = (i == 0) ? nx - 1 : i - 1;
    const long long r = (long long)j * nx, rn = r + nx;
    const long long c = r + i;
    E[c * 3 + 0] = 0.5 * (F.Ex[r + im] + F.Ex[r + i]);
    E[c * 3 + 1] = 0.5 * (F.Ey[r + i] + F.Ey[rn + i]);
    E[c * 3 + 2] = F.Ez[r + i];
    B[c * 3 + 0] = 0.5 * (F.Bx[r + i] + F.Bx[rn + i]);
    B[c * 3 + 1] = 0.5 * (F.By[r + im] + F.By[r + i]);
    const double lo = 0.5 * (F.Bz[r + im] + F.Bz[r + i]);
    const double hi = 0.5 * (F.Bz[rn + im] + F.Bz[rn + i]);
    B[c * 3 + 2] = 0.5 * (lo + hi);
}

// A whole half step from F to G (which must not overlap) in one launch, with
// the cell-centred averages the step takes from it: a block produces kFRows
// Yee rows x kFCols columns and holds what they depend on in shared memory (E
// two rows and columns beyond, B and the current one or two), so that the three
// updates run there.  As separate kernels a step's two half steps, averages and
// extrapolation are nine launches, of about 3 us each on a small grid, and at
// 1024 x 512 move every component four times (123 us; this 72).  Latency of the
// loads bounds it: 512 threads hold one point of each region, so all twelve loads
// of a thread are in flight at once (256 threads looping over the regions: 42 us
// at 1024 x 512, 11.4 at 256 x 128, 10 at 32 x 16; now 36, 6.7, 5.4).  Expressions
// and roundings are those of the kernels above: the velocity sweeps round the
// fields to FP32 coefficients, so a last-bit change here is not one there.
// Rows q of the tile are virtual: periodic y wraps them; between walls the
// integer-row components of E beyond a wall are minus their mirror image.
// With periodic y rows 0 and ny of the [ny+1] arrays are the same points but
// two copies, each advanced by itself: the integer rows beyond the seam take
// the copy on their own side (row ny below row 0, row 0 above row ny - 1).
constexpr int kFCols = 32, kFRows = 8, kHalfThreads = 512;
constexpr int kEC = kFCols + 4, kER = kFRows + 4;      // E: columns i0-2 .. i0+33, rows r0-2 .. r0+9
constexpr int kBC = kFCols + 3, kBR = kFRows + 3;      // B: columns i0-2 .. i0+32, rows r0-1 .. r0+9
constexpr int kJC = kFCols + 3, kJR = kFRows + 3;      // current: columns i0-1 .. i0+33, rows r0-2 .. r0+8

struct HalfArgs {
    YeeView F, G;
    Currents J;
    double hb, he, dx, dy;      // B -= hb curl E; E += he (curl B - j)
    // averages to cell centres (null: not wanted): of F, of G, and 2 G - F
    double *E0, *B0, *E1, *B1, *E2, *B2;
};

__global__ void __launch_bounds__(kHalfThreads) yee_half_kernel(HalfArgs A) {
    __shared__ double ex[kER][kEC], ey[kER][kEC], ez[kER][kEC];
    __shared__ double bx[kBR][kBC], by[kBR][kBC], bz[kBR][kBC];
    __shared__ double jx[kJR][kJC], jy[kJR][kJC], jz[kJR][kJC];
    __shared__ double eys[2][kEC], bxs[2][kBC], bzs[2][kBC];         // the seam's other copies: rows ny, 0
    const int nx = A.F.nx, ny = A.F.ny, per = A.F.per;
    const int i0 = (int)blockIdx.x * kFCols, r0 = (int)blockIdx.y * kFRows;
    const int tid = threadIdx.x;
    auto col = [nx](int i) {
        i %= nx;
        return i < 0 ? i + nx : i;
    };
    auto wrap = [ny](int q, int n) {          // periodic rows: the points of row q mod ny, in [0, n]
        while (q < 0) q += ny;
        while (q > n) q -= ny;
        return q;
    };
    // every load of a thread (one point of each region) in flight together: E's
    // rows of Ex, Ez outside [0, ny) by the boundary; rows no valid point needs are 0
    static_assert(kER * kEC <= kHalfThreads && kBR * kBC <= kHalfThreads && kJR * kJC <= kHalfThreads &&
                  2 * kEC <= kHalfThreads, "one point of each region per thread");
    const int re_ = min(tid / kEC, kER - 1), ce_ = tid % kEC;
    double sgn = 1.0;
    bool ok = true, okh = true;
    size_t at, ath;
    {
        const int i = col(i0 - 2 + ce_);
        int q = r0 - 2 + re_, h = q;
        if (per) {
            q = wrap(q, ny - 1);
            h = wrap(h, ny);
        } else {
            okh = q >= 0 && q <= ny;
            h = min(max(h, 0), ny);
            if (q < 0) {
                ok = q == -1;
                q = 0;
                sgn = -1.0;
            } else if (q >= ny) {
                ok = q == ny;
                q = ny - 1;
                sgn = -1.0;
            }
        }
        at = (size_t)q * nx + i;
        ath = (size_t)h * nx + i;
    }
    const double vex = A.F.Ex[at], vez = A.F.Ez[at], vey = A.F.Ey[ath];
    const int rb_ = min(tid / kBC, kBR - 1), cb_ = tid % kBC;
    bool bok = true, bokh = true;
    {
        const int i = col(i0 - 2 + cb_);
        int q = r0 - 1 + rb_, h = q;
        if (per) {
            q = wrap(q, ny - 1);
            h = wrap(h, ny);
        } else {
            bok = q >= 0 && q < ny;
            bokh = q >= 0 && q <= ny;
            h = min(max(h, 0), ny);
            q = min(max(q, 0), ny - 1);
        }
        at = (size_t)q * nx + i;
        ath = (size_t)h * nx + i;
    }
    const double vbx = A.F.Bx[ath], vbz = A.F.Bz[ath], vby = A.F.By[at];
    const int rj_ = min(tid / kJC, kJR - 1), cj_ = tid % kJC;
    bool jok = true;
    double m0[3] = {0.0, 0.0, 0.0}, m1[3] = {0.0, 0.0, 0.0};
    {
        int q = r0 - 2 + rj_;
        if (per) {
            q = wrap(q, ny - 1);
        } else {
            jok = q >= 0 && q < ny;
            q = min(max(q, 0), ny - 1);
        }
        const size_t cell = (size_t)q * nx + col(i0 - 1 + cj_);
        if (A.J.ns > 0) {
            const double* m = A.J.mom[0] + cell * A.J.stride + 1;
#pragma unroll
            for (int d = 0; d < 3; ++d) m0[d] = m[d];
        }
        if (A.J.ns > 1) {
            const double* m = A.J.mom[1] + cell * A.J.stride + 1;
#pragma unroll
            for (int d = 0; d < 3; ++d) m1[d] = m[d];
        }
    }
    // the seam in this tile: row 0 at virtual row 0, and row ny
    const bool seam[2] = {per && r0 == 0, per && r0 + kFRows + 1 >= ny};
    if (per && tid < 2 * kEC) {
        const int s = tid / kEC, c = tid % kEC;
        const size_t as = (s == 0 ? (size_t)ny * nx : 0) + col(i0 - 2 + c);
        if (seam[s]) {
            eys[s][c] = A.F.Ey[as];
            if (c < kBC) {
                bxs[s][c] = A.F.Bx[as];
                bzs[s][c] = A.F.Bz[as];
            }
        }
    }
    if (tid < kER * kEC) {
        ex[re_][ce_] = ok ? sgn * vex : 0.0;
        ez[re_][ce_] = ok ? sgn * vez : 0.0;
        ey[re_][ce_] = okh ? vey : 0.0;
    }
    if (tid < kBR * kBC) {
        bx[rb_][cb_] = bokh ? vbx : 0.0;
        bz[rb_][cb_] = bokh ? vbz : 0.0;
        by[rb_][cb_] = bok ? vby : 0.0;
    }
    if (tid < kJR * kJC) {
        double v[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            v[d] = A.J.ns > 0 ? fma(A.J.q[0], m0[d], 0.0) : 0.0;
            if (A.J.ns > 1) v[d] = fma(A.J.q[1], m1[d], v[d]);
            if (!jok) v[d] = 0.0;
        }
        jx[rj_][cj_] = v[0];
        jy[rj_][cj_] = v[1];
        jz[rj_][cj_] = v[2];
    }
    __syncthreads();
    // this thread's point: column i0 + tc, row r0 + tr
    const int tc = tid % kFCols, tr = tid / kFCols;
    const int i = i0 + tc, q = r0 + tr;
    const bool point = tid < kFRows * kFCols && i < nx, cell = point && q < ny;
    // averages at the cell (E arrays start two rows and columns before the tile, B arrays one row and two columns)
    auto averages = [&](double (&e)[3], double (&b)[3]) {
        const int re = tr + 2, rb = tr + 1, c = tc + 2;
        e[0] = 0.5 * (ex[re][c - 1] + ex[re][c]);
        e[1] = 0.5 * (ey[re][c] + ey[re + 1][c]);
        e[2] = ez[re][c];
        b[0] = 0.5 * (bx[rb][c] + bx[rb + 1][c]);
        b[1] = 0.5 * (by[rb][c - 1] + by[rb][c]);
        const double lo = 0.5 * (bz[rb][c - 1] + bz[rb][c]);
        const double hi = 0.5 * (bz[rb + 1][c - 1] + bz[rb + 1][c]);
        b[2] = 0.5 * (lo + hi);
    };
    double e0[3] = {0.0, 0.0, 0.0}, b0[3] = {0.0, 0.0, 0.0};
    const size_t at3 = ((size_t)q * nx + i) * 3;
    if (A.E0 && cell) {
        averages(e0, b0);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            A.E0[at3 + d] = e0[d];
            A.B0[at3 + d] = b0[d];
        }
    }
    __syncthreads();
    // B -= hb curl E on the whole B region (B row r is E row r + 1)
    auto curl_e = [&](int r, int c) {
        const double dEz = (ez[r + 1][c] - ez[r][c]) / A.dy;
        const double dEy = (ey[r + 1][c + 1] - ey[r + 1][c]) / A.dx, dEx = (ex[r + 1][c] - ex[r][c]) / A.dy;
        bx[r][c] = fma(-A.hb, dEz, bx[r][c]);
        bz[r][c] = fma(-A.hb, dEy - dEx, bz[r][c]);
        by[r][c] = by[r][c] + A.hb * (ez[r + 1][c + 1] - ez[r + 1][c]) / A.dx;
    };
    if (tid < kBR * kBC) curl_e(tid / kBC, tid % kBC);
    if (per) {
        const int s = tid / kBC, c = tid % kBC;
        if (s < 2 && seam[s]) {
            const int re = (s == 0 ? 0 : ny) - (r0 - 2);
            const double dEz = (ez[re][c] - ez[re - 1][c]) / A.dy;
            const double dEy = (eys[s][c + 1] - eys[s][c]) / A.dx, dEx = (ex[re][c] - ex[re - 1][c]) / A.dy;
            bxs[s][c] = fma(-A.hb, dEz, bxs[s][c]);
            bzs[s][c] = fma(-A.hb, dEy - dEx, bzs[s][c]);
        }
    }
    __syncthreads();
    // E += he (curl B - j) on rows r0-1 .. r0+8, columns i0-1 .. i0+32
    if (tid < (kFRows + 2) * (kFCols + 2)) {
        const int r = tid / (kFCols + 2) + 1, c = tid % (kFCols + 2) + 1;     // in the E arrays
        const int rb = r - 1, rj = r, cj = c - 1;
        const int row = r0 - 2 + r;
        const bool below = per && row == -1, above = per && row == ny;
        const double bzl = above ? bzs[1][c] : bz[rb][c], bzh = below ? bzs[0][c] : bz[rb + 1][c];
        const double bxl = above ? bxs[1][c] : bx[rb][c], bxh = below ? bxs[0][c] : bx[rb + 1][c];
        const double cx = (bzh - bzl) / A.dy - 0.5 * (jx[rj][cj] + jx[rj][cj + 1]);
        const bool wall = !per && (row == 0 || row == ny);
        const double cy = -(bz[rb][c] - bz[rb][c - 1]) / A.dx - (wall ? 0.0 : 0.5 * (jy[rj - 1][cj] + jy[rj][cj]));
        const double cz = (by[rb][c] - by[rb][c - 1]) / A.dx - (bxh - bxl) / A.dy - jz[rj][cj];
        ex[r][c] = fma(A.he, cx, ex[r][c]);
        ey[r][c] = fma(A.he, cy, ey[r][c]);
        ez[r][c] = fma(A.he, cz, ez[r][c]);
    }
    __syncthreads();
    if (!per) {        // ghost rows -1 and ny mirror rows 0 and ny - 1
        if (tid < 2 * (kFCols + 2)) {
            const int c = tid % (kFCols + 2) + 1;
            const int g = (tid < kFCols + 2 ? -1 : ny) - (r0 - 2), m = (tid < kFCols + 2 ? 0 : ny - 1) - (r0 - 2);
            if (g >= 1 && g <= kFRows + 2 && m >= 1 && m <= kFRows + 2) {
                ex[g][c] = -ex[m][c];
                ez[g][c] = -ez[m][c];
            }
        }
        __syncthreads();
    }
    // B -= hb curl E on rows r0 .. r0+8, columns i0-1 .. i0+31
    if (tid < (kFRows + 1) * (kFCols + 1)) curl_e(tid / (kFCols + 1) + 1, tid % (kFCols + 1) + 1);
    __syncthreads();
    if (point && q <= ny) {
        const size_t at = (size_t)q * nx + i;
        const int re = tr + 2, rb = tr + 1, c = tc + 2;
        A.G.Ey[at] = ey[re][c];
        A.G.Bx[at] = bx[rb][c];
        A.G.Bz[at] = bz[rb][c];
        if (q < ny) {
            A.G.Ex[at] = ex[re][c];
            A.G.Ez[at] = ez[re][c];
            A.G.By[at] = by[rb][c];
        }
    }
    if (A.E1 && cell) {
        double e1[3], b1[3];
        averages(e1, b1);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            A.E1[at3 + d] = e1[d];
            A.B1[at3 + d] = b1[d];
            if (A.E2) {
                A.E2[at3 + d] = 2.0 * e1[d] - e0[d];
                A.B2[at3 + d] = 2.0 * b1[d] - b0[d];
            }
        }
    }
}

// The B-curl kernel reads the current from the species' moment records (8-byte
// lanes 80 or 160 bytes apart, several records per lane): dynamic LDS that it
// does not use caps it at eight one-wave blocks per CU (two waves per SIMD),
// so fewer waves evict the lines those loads share.  2048 x 1024 cells: the
// three half-step kernels 0.74 -> 0.50 ms per fluid-only step (one wave per
// SIMD 0.63, three 0.49, four 0.66).
constexpr unsigned kCurlBLdsCap = 20480;

hipError_t launch_maxwell_half(double* yee, int nx, int ny, const double* const* mom, const double* q, int ns,
                               double dt, double c, double dx, double dy, hipStream_t st, int mstride, int per) {
    YeeView F = yee_view(yee, nx, ny);
    F.per = per;
    Currents J;
    J.ns = ns;
    J.stride = mstride;
    for (int k = 0; k < 2; ++k) {
        J.mom[k] = k < ns ? mom[k] : nullptr;
        J.q[k] = k < ns ? q[k] : 0.0;
    }
    const double h = 0.5 * dt;
    dim3 blk(64), grid((nx + 63) / 64, ny + 1);
    hipLaunchKernelGGL(yee_curl_e_kernel, grid, blk, 0, st, F, 0.5 * h, dx, dy);
    hipLaunchKernelGGL(yee_curl_b_kernel, grid, blk, kCurlBLdsCap, st, F, J, h, c * c, dx, dy);
    hipLaunchKernelGGL(yee_curl_e_kernel, grid, blk, 0, st, F, 0.5 * h, dx, dy);
    return hipGetLastError();
}

hipError_t launch_cell_fields(const double* yee, int nx, int ny, double* E, double* B, hipStream_t st) {
    YeeView F = yee_view(const_cast<double*>(yee), nx, ny);
    hipLaunchKernelGGL(cell_fields_kernel, dim3((nx + 63) / 64, ny), dim3(64), 0, st, F, E, B);
    return hipGetLastError();
}

hipError_t launch_yee_half(const double* from, double* to, int nx, int ny, const double* const* mom, const double* q,
                           int ns, double dt, double c, double dx, double dy, int mstride, int per,
                           const CellFields& at_from, const CellFields& at_to, const CellFields& ahead,
                           hipStream_t st) {
    HalfArgs A;
    A.F = yee_view(const_cast<double*>(from), nx, ny);
    A.G = yee_view(to, nx, ny);
    A.F.per = A.G.per = per;
    A.J.ns = ns;
    A.J.stride = mstride;
    for (int k = 0; k < 2; ++k) {
        A.J.mom[k] = k < ns ? mom[k] : nullptr;
        A.J.q[k] = k < ns ? q[k] : 0.0;
    }
    const double h = 0.5 * dt;
    A.hb = 0.5 * h;
    A.he = h * (c * c);
    A.dx = dx;
    A.dy = dy;
    A.E0 = at_from.E;
    A.B0 = at_from.B;
    A.E1 = at_to.E;
    A.B1 = at_to.B;
    A.E2 = ahead.E;
    A.B2 = ahead.B;
    hipLaunchKernelGGL(yee_half_kernel, dim3((nx + kFCols - 1) / kFCols, (ny + kFRows) / kFRows), dim3(kHalfThreads), 0, st, A);
    return hipGetLastError();
}

// Field energy, deterministic: block partials over the rows jh = 0..ny (one
// block column per row, fixed order), then one block adds them.
// 2X3V: sum of B^2/2 + E^2/(2 c^2) over the Yee points, wall rows of the
// [ny+1] arrays (Ey, Bx, Bz) at half weight; 1X1V: sum of E^2/2.
__global__ void __launch_bounds__(256)
field_energy_rows_kernel(YeeView F, double inv_c2, double* __restrict__ part) {
    __shared__ double red[4];
    const int jh = blockIdx.x;
    const int nx = F.nx, ny = F.ny;
    double acc[1] = {0.0};
    const double w = (jh == 0 || jh == ny) ? 0.5 : 1.0;
    const long long h = (long long)jh * nx;
    for (int i = threadIdx.x; i < nx; i += blockDim.x) {
        double e = w * (F.Bx[h + i] * F.Bx[h + i] + F.Bz[h + i] * F.Bz[h + i] + inv_c2 * F.Ey[h + i] * F.Ey[h + i]);
        if (jh < ny) e += F.By[h + i] * F.By[h + i] + inv_c2 * (F.Ex[h + i] * F.Ex[h + i] + F.Ez[h + i] * F.Ez[h + i]);
        acc[0] += 0.5 * e;
    }
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) part[jh] = acc[0];
}

__global__ void __launch_bounds__(256)
line_energy_kernel(const double* __restrict__ E, int n, double* __restrict__ part) {
    __shared__ double red[4];
    double acc[1] = {0.0};
    for (int i = threadIdx.x; i < n; i += blockDim.x) acc[0] += 0.5 * E[i] * E[i];
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) part[0] = acc[0];
}

__global__ void __launch_bounds__(256)
ordered_sum_kernel(const double* __restrict__ part, int np, double scale, double* __restrict__ out) {
    __shared__ double red[4];
    // thread t adds partials t, t+256, ... in order; then a fixed-order block sum
    double acc[1] = {0.0};
    for (int i = threadIdx.x; i < np; i += blockDim.x) acc[0] += part[i];
    block_sum<1>(acc, red);
    if (threadIdx.x == 0) *out = acc[0] * scale;
}

hipError_t launch_field_energy(const double* fields, int dim_x, int nx, int ny, double c, double dX, double* part,
                               double* out, hipStream_t st) {
    if (dim_x == 2) {
        const YeeView F = yee_view(const_cast<double*>(fields), nx, ny);
        hipLaunchKernelGGL(field_energy_rows_kernel, dim3(ny + 1), dim3(256), 0, st, F, 1.0 / (c * c), part);
        hipLaunchKernelGGL(ordered_sum_kernel, dim3(1), dim3(256), 0, st, part, ny + 1, dX, out);
    } else {
        hipLaunchKernelGGL(line_energy_kernel, dim3(1), dim3(256), 0, st, fields, nx, part);
        hipLaunchKernelGGL(ordered_sum_kernel, dim3(1), dim3(256), 0, st, part, 1, dX, out);
    }
    return hipGetLastError();
}

}  // namespace vl
