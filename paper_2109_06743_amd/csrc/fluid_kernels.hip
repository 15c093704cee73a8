// Ten-moment fluid step for gfx950 (FP64): Eqs. 2-4 of arXiv 2109.06743 with
// the flux of the second moment P given by the third moment Qcal taken from f
// (Algorithm 1).  Semi-discrete finite volumes: CWENO-3 (Kurganov-Levy)
// point values at the faces, local Lax-Friedrichs flux with speed
// |u_d| + sqrt(3 p_dd / (m n)), and SSP-RK3 (Shu-Osher) in time.
//
// One launch per RK stage does all of it for every species: third moment (from
// f, or a closure of the stage state), face fluxes of both directions,
// L(U) = -div H + S(U, E, B) and the stage combination
// U_out = a U_n + b (U_s + dt L).
//
// Component orders: U = (n, nu_x, nu_y, nu_z, Pxx, Pxy, Pxz, Pyy, Pyz, Pzz);
// Qcal (from the raw moment vector, offset 10) = (xxx, xxy, xxz, xyy, xyz,
// xzz, yyy, yyz, yzz, zzz).  1V: U = (n, nu, P), Qcal = raw moment 3.
#include "vl_internal.h"

// Every rounding here is written out: multiply-adds are fused where fma() says
// so and nowhere else, quotients are correctly rounded.  The fit rounds
// functions of U to the type of f, where a last bit of U can become one of f's,
// so U must not depend on how a kernel is split or optimised: a network closure
// that falls back gives the kinetic step bit for bit, and the tests form the
// same roundings on the host.
#pragma clang fp contract(off)

namespace vl {

constexpr double kCwenoEps = 1e-6;

// Quotients by one divisor, bit for bit those of `/` while no step leaves the
// normal numbers (divisors up to 2^1021, numerators from 2^-968; zeros,
// infinities and NaN as `/`): the hardware's estimate of 1/x, two Newton steps
// and a correction of each quotient by its remainder.  What `/` does besides is
// to scale its operands, and to form 1/x again for every numerator.
struct Divisor {
    double x, r;
    __device__ __forceinline__ explicit Divisor(double v) : x(v) {
        r = __builtin_amdgcn_rcp(x);
        r = fma(fma(-x, r, 1.0), r, r);
        r = fma(fma(-x, r, 1.0), r, r);
    }
    __device__ __forceinline__ double under(double a) const {
        const double q = a * r;
        return __builtin_amdgcn_div_fixup(fma(fma(-x, q, a), r, q), x, a);
    }
};

// CWENO-3 point values of cell j at its left (x_j - h/2) and right (x_j + h/2)
// faces from the averages a = u_{j-1}, b = u_j, c = u_{j+1}.  The left, right
// and centred polynomials evaluated at +-h/2 are
//   P_L = b -+ (b - a)/2,  P_R = b -+ (c - b)/2,  P_C = b + d2/6 -+ (c - a)/4,
// d2 = c - 2b + a, weighted with (1/4, 1/2, 1/4) / (eps + IS)^2, normalised.
// With D = (eps + IS)^2 the normalised weights are
//   w_L = Dc Dr / S, w_C = 2 Dl Dr / S, w_R = Dl Dc / S,
//   S = Dc Dr + 2 Dl Dr + Dl Dc
// (one division), and since they sum to one the point values are b plus the
// weighted corrections (a constant state reconstructs to itself exactly), here
// b + 1/2 (w_C d2/3 +- (w_L (b-a) + w_R (c-b) + w_C (c-a)/2)).  39 operations;
// the reconstructions are two thirds of the stage kernel's arithmetic.
__device__ __forceinline__ void cweno(double a, double b, double c, double& left, double& right) {
    const double dl = b - a, dr = c - b, d2 = fma(-2.0, b, c) + a, hc = 0.5 * (c - a);
    const double el = fma(dl, dl, kCwenoEps), er = fma(dr, dr, kCwenoEps);
    const double ec = fma(hc, hc, fma(d2, d2 * (13.0 / 3.0), kCwenoEps));
    const double Dl = el * el, Dc = ec * ec, Dr = er * er, Dl2 = Dl + Dl;
    const double tl = Dc * Dr, tc = Dl2 * Dr, tr = Dl * Dc;
    const double inv = Divisor(fma(Dl, Dc, fma(Dl2, Dr, tl))).under(1.0);
    const double wl = tl * inv, wc = tc * inv, wr = tr * inv;
    const double side = fma(hc, wc, fma(dl, wl, dr * wr));           // twice the odd part
    const double even = d2 * (1.0 / 3.0);                            // twice the even part: even wc
    right = fma(0.5, fma(even, wc, side), b);
    left = fma(0.5, fma(even, wc, -side), b);
}

// y-parity (+1/-1) of U and Qcal components under y -> -y
__device__ __forceinline__ double par_u(int k) {
    return (k == 2 || k == 5 || k == 8) ? -1.0 : 1.0;       // nu_y, Pxy, Pyz
}
__device__ __forceinline__ double par_q(int k) {
    return (k == 1 || k == 4 || k == 6 || k == 8) ? -1.0 : 1.0;  // xxy, xyz, yyy, yzz
}

// Value of lane + 1 (kUp) or lane - 1 of the same 16-lane row.
template <bool kUp>
__device__ __forceinline__ double row_next(double v) {
    constexpr int ctrl = kUp ? 0x101 : 0x111;               // row_shl:1, row_shr:1
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// One RK stage of the ten-moment fluid.  A 512-thread block updates kRows x
// kCols cells; its first half takes the x direction and the sources, its
// second half the y direction:
// 1. U (first half) and the kinetic third moment (second half) of the cells
//    and two more on each side go to shared memory, one array per component,
//    in runs of 180 consecutive doubles per row (wrapped in x, mirrored or
//    wrapped in y); with a closure the block forms the third moments there.
// 2. x: 16 lanes per row, the outer two for the neighbour cells; each lane
//    reconstructs its cell (16 components: U and the six third moments with an
//    x index), takes the next cell's lower point values from the next lane and
//    forms the flux through its upper face; the flux through its lower face is
//    the previous lane's.
// 3. y: the same for kRows + 2 rows, through shared memory (which no longer
//    holds the cells).
// 4. The first half adds both and the second writes rows of 140 doubles.
// The kernel is bound by its FP64 instructions (two thirds of them in cweno).
// Two kernels per stage used to store the fluxes (160 B a cell) and read them
// back from 80-byte records, reconstruct all 20 components per direction and,
// with a closure, read and write a third moment (2 x 160 B) and an Eq. 5
// source first: 125 + 63 + 25 + 22 us a stage at 1024 x 512, one species; this
// takes 71 (Eq. 5), and 11.4 us instead of 6.6 + 4.1 on 32 x 16 cells (both
// species), with the same bits.  Estimated reciprocals in place of the quotients
// and the two differences added to U one after the other took 65 and 10.9, but
// changed the bits of U, and in a magnetotail step about one cell in ten million
// then got another FP32 distribution, by 6e-8.
enum { kThirdKinetic = 0, kThirdZero = 1, kThirdNet = 2 };
constexpr int kRows = 16, kCols = 14;
constexpr int kHaloR = kRows + 4, kHaloC = kCols + 4;
constexpr int kHaloCells = kHaloR * kHaloC;
constexpr int kStageComps = 19;               // U and Qcal without zzz, which no flux takes
constexpr int kXLanes = kRows * (kCols + 2), kYLanes = (kRows + 2) * kCols;
constexpr int kHalf = 256;                    // threads per direction
constexpr int kTempCells = (kRows + 2) * (kCols + 2);
constexpr int kXStride = kXLanes + 1, kYStride = kYLanes + 1;    // of the exchange arrays
static_assert(kXLanes <= kHalf && kYLanes <= kHalf && kHaloC * 10 <= kHalf, "one pass each");
static_assert(17 * kYStride <= kStageComps * kHaloCells, "the y exchange fits the cells' memory");
static_assert(kRows * kCols * 10 <= 10 * kYStride, "the results fit the y fluxes' memory");
static_assert(10 * (kXStride + kYStride) <= kStageComps * kHaloCells, "fluxes and differences fit the cells' memory");

struct FluidArgs {
    int nx, ny;
    double idx, idy;      // 1/dx, 1/dy
    double a, b, dt;      // stage: Uo = a Un + b (Us + dt L)
    double wa, wb;        // kinetic third moment wa QA + wb QB
    const double* E;      // [cells][3]
    const double* B;
    int per;              // 1: periodic y, 0: reflecting walls
    int tx, ty;           // tiles along x, y
};

// Third moment u_a P_bc + u_b P_ac + u_c P_ab - 2 m n u_a u_b u_c + heat[k], for
// component k of nine (heat: the closure's heat flux, sc y in kNet's terms).
template <class Heat>
__device__ __forceinline__ void third_moment(const double (&U)[10], const double (&u)[3], double m, double (&Q)[9],
                                             const Heat& heat) {
    const double mn2 = 2.0 * m * U[0];
    const double P[3][3] = {{U[4], U[5], U[6]}, {U[5], U[7], U[8]}, {U[6], U[8], U[9]}};
    const int ta[9] = {0, 0, 0, 0, 0, 0, 1, 1, 1}, tb[9] = {0, 0, 0, 1, 1, 2, 1, 1, 2}, tc[9] = {0, 1, 2, 1, 2, 2, 1, 2, 2};
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int x = ta[k], y = tb[k], z = tc[k];
        const double first = u[y] * P[x][z];
        const double two = x == y ? first + first : fma(u[x], P[y][z], first);
        const double three = heat(k, fma(u[z], P[x][y], two));
        Q[k] = fma(-(mn2 * u[x] * u[y]), u[z], three);
    }
}

// Temperature tensor T = (P - m n u u) / n of a fluid record (PAIRS order).
__device__ __forceinline__ void temperature6(const double (&V)[10], const double (&u)[3], const Divisor& n, double m,
                                             double (&T)[6]) {
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
    const double mn = m * V[0];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double mnu = mn * u[pa[k]], ub = u[pb[k]];
        T[k] = n.under(k == 1 || k == 4 ? V[4 + k] - mnu * ub : fma(-mnu, ub, V[4 + k]));
    }
}

// Face fluxes of one direction: W components 0..9 are U, 10..15 the third
// moments of the second-moment fluxes in PAIRS order; src[k] the component
// whose value is flux k (n -> nu_d, nu_i -> P_id / m, P_ab -> Qcal_abd).
template <int D>
struct FluxMap {
    // raw component of W[10 + k]: Qcal_abd of the pair ab
    static __device__ __forceinline__ constexpr int third(int k) {
        constexpr int x[6] = {0, 1, 2, 3, 4, 5}, y[6] = {1, 3, 4, 6, 7, 8};
        return 10 + (D == 0 ? x[k] : y[k]);
    }
    static __device__ __forceinline__ constexpr int src(int k) {
        constexpr int x[10] = {1, 4, 5, 6, 10, 11, 12, 13, 14, 15};
        constexpr int y[10] = {2, 5, 7, 8, 10, 11, 12, 13, 14, 15};
        return D == 0 ? x[k] : y[k];
    }
    static constexpr int nu = 1 + D, pdd = D == 0 ? 4 : 7;
};

template <int D>
__device__ __forceinline__ double wave_speed(const double (&W)[16], double m) {
    const double u = W[FluxMap<D>::nu] / W[0], mn = m * W[0];
    const double p = fma(-u, mn * u, W[FluxMap<D>::pdd]);
    return fabs(u) + sqrt(fmax(3.0 * p / mn, 0.0));
}

// Local Lax-Friedrichs flux k between the point values Wm (below) and Wp; ha:
// half the wave speed.
template <int D>
__device__ __forceinline__ double face_flux(const double (&Wm)[16], const double (&Wp)[16], int k, double ha, double im) {
    const double fm = Wm[FluxMap<D>::src(k)], fp = Wp[FluxMap<D>::src(k)];
    const double sum = k >= 1 && k < 4 ? fma(im, fm, im * fp) : fp + fm;
    return fma(0.5, sum, -(ha * (Wp[k] - Wm[k])));
}

template <int THIRD>
__global__ void __launch_bounds__(2 * kHalf) __attribute__((amdgpu_waves_per_eu(4)))
fluid3_stage_kernel(FluidSet S, FluidArgs A) {
    __shared__ double raw[kStageComps][kHaloCells];
    double* const pool = &raw[0][0];
    double* const part = pool + 10 * kYStride;   // y differences, next to the y fluxes
    __shared__ double temp[THIRD == kThirdZero ? 6 * kTempCells : 1];
    const unsigned per_sp = (unsigned)(A.tx * A.ty);
    const unsigned w = xcd_work_index(blockIdx.x, gridDim.x);
    const int sp = (int)(w / per_sp);
    const int i0 = (int)(w % per_sp % (unsigned)A.tx) * kCols, j0 = (int)(w % per_sp / (unsigned)A.tx) * kRows;
    const double* __restrict__ Us = S.Us[sp];
    const double m = S.m[sp], q = S.q[sp];
    const int nx = A.nx, ny = A.ny;
    const bool xhalf = threadIdx.x < kHalf;                 // wave-uniform
    const int tid = threadIdx.x & (kHalf - 1);

    // row of a halo row: itself, ~row where mirrored, kNoRow where no flux
    // needs it (lane = halo row; the loops read it back per row)
    constexpr int kNoRow = -0x7fffffff;
    auto map_row = [&](int j) {
        if (A.per) {
            j %= ny;
            return j < 0 ? j + ny : j;
        }
        if (j < 0) return ~(-1 - j);
        if (j < ny) return j;
        return j <= ny + 1 ? ~(2 * ny - 1 - j) : kNoRow;
    };
    auto source_of = [](int row) { return row == kNoRow ? 0 : (row < 0 ? ~row : row); };
    auto col_of_i = [&](int i) {
        i %= nx;
        return i < 0 ? i + nx : i;
    };
    const int rows_v = map_row(j0 - 2 + (tid & 31));
    const bool mirrored = !A.per && (j0 < 2 || j0 + kRows + 2 > ny);
    // 1. cells and ring: all the loads of a thread in flight together
    const bool kinetic = THIRD == kThirdKinetic || (THIRD == kThirdNet && S.fallback[sp] && *S.fallback[sp]);
    if (tid < kHaloC * 10 && (xhalf || kinetic)) {
        const int l = tid / 10, k = tid % 10;
        const unsigned i = (unsigned)col_of_i(i0 - 2 + l);
        double v[kHaloR];
        if (xhalf) {
#pragma unroll
            for (int jj = 0; jj < kHaloR; ++jj) {
                const double* row = Us + (size_t)source_of(__builtin_amdgcn_readlane(rows_v, jj)) * nx * 10;
                v[jj] = row[i * 10u + (unsigned)k];
            }
            if (mirrored) {
                const double su = par_u(k);
#pragma unroll
                for (int jj = 0; jj < kHaloR; ++jj)
                    if (__builtin_amdgcn_readlane(rows_v, jj) < 0) v[jj] *= su;
            }
#pragma unroll
            for (int jj = 0; jj < kHaloR; ++jj) raw[k][jj * kHaloC + l] = v[jj];
        } else if (k < 9) {
            const double* __restrict__ QA = S.QA[sp];
            const double* __restrict__ QB = S.QB[sp];
#pragma unroll
            for (int jj = 0; jj < kHaloR; ++jj) {
                const double* row = QA + (size_t)source_of(__builtin_amdgcn_readlane(rows_v, jj)) * nx * 20;
                v[jj] = A.wa * row[i * 20u + 10u + (unsigned)k];
            }
            if (A.wb != 0.0) {
#pragma unroll
                for (int jj = 0; jj < kHaloR; ++jj) {
                    const double* row = QB + (size_t)source_of(__builtin_amdgcn_readlane(rows_v, jj)) * nx * 20;
                    v[jj] = fma(A.wb, row[i * 20u + 10u + (unsigned)k], v[jj]);
                }
            }
            if (mirrored) {
                const double sq = par_q(k);
#pragma unroll
                for (int jj = 0; jj < kHaloR; ++jj)
                    if (__builtin_amdgcn_readlane(rows_v, jj) < 0) v[jj] *= sq;
            }
#pragma unroll
            for (int jj = 0; jj < kHaloR; ++jj) raw[10 + k][jj * kHaloC + l] = v[jj];
        }
    }
    __syncthreads();
    if (THIRD != kThirdKinetic && !kinetic) {
        // third moments of the cross of cells that fluxes need: kRows full rows,
        // and two rows above and below without the outer columns
        const int e = (int)threadIdx.x, f = e - kRows * kHaloC;
        if (f < 4 * kCols) {
            const int jj = f < 0 ? e / kHaloC + 2 : (f / kCols < 2 ? f / kCols : f / kCols + kRows);
            const int l = f < 0 ? e % kHaloC : f % kCols + 2;
            const int c = jj * kHaloC + l;
            double V[10], Q[9];
#pragma unroll
            for (int k = 0; k < 10; ++k) V[k] = raw[k][c];
            const Divisor n(V[0]);
            const double u[3] = {n.under(V[1]), n.under(V[2]), n.under(V[3])};
            if (THIRD == kThirdNet) {
                const int row = map_row(j0 - 2 + jj);
                const long long g = (long long)source_of(row) * nx + col_of_i(i0 - 2 + l);
                const double sc = S.scale[sp][g];
                const float* __restrict__ y = S.y[sp] + g * 16;
                third_moment(V, u, m, Q, [&](int k, double v) {
                    return fma(row < 0 ? sc * par_q(k) : sc, (double)y[k], v);
                });
            } else {
                third_moment(V, u, m, Q, [](int, double v) { return v; });
            }
#pragma unroll
            for (int k = 0; k < 9; ++k) raw[10 + k][c] = Q[k];
            if (THIRD == kThirdZero && l >= 1 && l <= kCols + 2 && jj >= 1 && jj <= kRows + 2) {
                double T[6];
                temperature6(V, u, n, m, T);
#pragma unroll
                for (int k = 0; k < 6; ++k) temp[k * kTempCells + (jj - 1) * (kCols + 2) + l - 1] = T[k];
            }
        }
        __syncthreads();
    }
    // reconstructions the scheduler may interleave (all 16 spill)
    constexpr int kBatch = 4;
    const double im = 1.0 / m;
    if (xhalf) {
        // 2. x
        const int tx = tid & (kCols + 1), ty = tid / (kCols + 2);
        const int r = (ty + 2) * kHaloC + tx + 1;
        const int i = i0 - 1 + tx, j = j0 + ty;
        const bool own = tx > 0 && tx <= kCols && i < nx && j < ny;
        double u[10], D[10], L[10];           // L: sources, D: x differences of the fluxes
        {
            double lo[16], hi[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int c = k < 10 ? k : FluxMap<0>::third(k - 10);
                cweno(raw[c][r - 1], raw[c][r], raw[c][r + 1], lo[k], hi[k]);
                if (k % kBatch == kBatch - 1) __builtin_amdgcn_sched_barrier(0);
            }
            const double slo = wave_speed<0>(lo, m), shi = wave_speed<0>(hi, m);
            const double ha = 0.5 * fmax(shi, row_next<true>(slo));
#pragma unroll
            for (int k = 0; k < 16; ++k) lo[k] = row_next<true>(lo[k]);
#pragma unroll
            for (int k = 0; k < 10; ++k) {
                const double H = face_flux<0>(hi, lo, k, ha, im);
                D[k] = H - row_next<false>(H);
            }
        }
        double Ev[3] = {0.0, 0.0, 0.0}, Bv[3] = {0.0, 0.0, 0.0};
        if (own) {
            const size_t c = ((size_t)j * nx + i) * 3;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                Ev[d] = A.E[c + d];
                Bv[d] = A.B[c + d];
            }
        }
#pragma unroll
        for (int k = 0; k < 10; ++k) u[k] = raw[k][r];
        __syncthreads();                      // every read of the cells is done
        // sources: momentum (q/m)(n E + nu x B), the factor q/m below
        const double qm = q / m;
        L[1] = fma(-u[3], Bv[1], fma(Ev[0], u[0], Bv[2] * u[2]));
        L[2] = fma(-u[1], Bv[2], fma(Ev[1], u[0], Bv[0] * u[3]));
        L[3] = fma(-u[2], Bv[0], fma(Ev[2], u[0], Bv[1] * u[1]));
        // second moment: q (nu_i E_j + nu_j E_i) + (q/m)(eps_jkl P_ik B_l + eps_ikl P_jk B_l)
        const double P[3][3] = {{u[4], u[5], u[6]}, {u[5], u[7], u[8]}, {u[6], u[8], u[9]}};
        double PxB[3][3];                     // row i of P crossed with B
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            PxB[d][0] = d == 0 ? fma(-Bv[1], P[d][2], Bv[2] * P[d][1]) : fma(P[d][1], Bv[2], -(P[d][2] * Bv[1]));
            PxB[d][1] = fma(P[d][2], Bv[0], -(P[d][0] * Bv[2]));
            PxB[d][2] = fma(P[d][0], Bv[1], -(P[d][1] * Bv[0]));
        }
        const int ia[6] = {0, 0, 0, 1, 1, 2}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int x = ia[k], y = ib[k];
            const double nE = u[1 + y] * Ev[x];
            L[4 + k] = fma(q, x == y ? nE + nE : fma(u[1 + x], Ev[y], nE), qm * (PxB[x][y] + PxB[y][x]));
        }
        __syncthreads();                      // the y exchange is stored
        double G[6];
        if constexpr (THIRD == kThirdZero) {
            // Eq. 5 as a source of P: -div Q = gchi n v_t lap T (gchi = chi / k0)
            if (own) {
                const double* t = temp + (ty + 1) * (kCols + 2) + tx;
                const double tr = t[0] + t[3 * kTempCells] + t[5 * kTempCells];
                const double g = S.gchi[sp] * (u[0] * sqrt(tr / (3.0 * m)));
                const double ix2 = A.idx * A.idx, iy2 = A.idy * A.idy;
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const double* tk = t + k * kTempCells;
                    const double lx = fma(-2.0, tk[0], tk[1]) + tk[-1];
                    const double ly = fma(-2.0, tk[0], tk[kCols + 2]) + tk[-(kCols + 2)];
                    G[k] = g * fma(lx, ix2, ly * iy2);
                }
            }
        }
        __syncthreads();                      // the y exchange has been read
        __syncthreads();                      // the y fluxes are stored
        __syncthreads();                      // the y differences are stored
        // 4. both directions
        if (own) {
            double* out = pool + (ty * kCols + tx - 1) * 10;
#pragma unroll
            for (int k = 0; k < 10; ++k) {
                const double d = fma(A.idx, D[k], part[k * kXStride + tid]);
                double l = k == 0 ? -d : (k < 4 ? fma(qm, L[k], -d) : L[k] - d);
                if constexpr (THIRD == kThirdZero)
                    if (k >= 4) l += G[k - 4];
                out[k] = fma(A.dt, l, u[k]);
            }
        }
        __syncthreads();                      // the results are stored
    } else {
        // 3. y
        const bool lane = tid < kYLanes;
        const int t = lane ? tid : 0;
        // lanes without a cell store into the padding entry: behind a branch the
        // compiler would move part of every reconstruction, and its inputs spill
        const int ts = lane ? tid : kYLanes;
        const int tx = t % kCols, ty = t / kCols;
        const int r = (ty + 1) * kHaloC + tx + 2;
        double lo[16], hi[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int c = k < 10 ? k : FluxMap<1>::third(k - 10);
            cweno(raw[c][r - kHaloC], raw[c][r], raw[c][r + kHaloC], lo[k], hi[k]);
            if (k % kBatch == kBatch - 1) __builtin_amdgcn_sched_barrier(0);
        }
        const double slo = wave_speed<1>(lo, m), shi = wave_speed<1>(hi, m);
        __syncthreads();                      // every read of the cells is done
#pragma unroll
        for (int k = 0; k < 16; ++k) pool[k * kYStride + ts] = lo[k];
        pool[16 * kYStride + ts] = slo;
        __syncthreads();                      // the y exchange is stored
        const int up = ty <= kRows ? t + kCols : t;
#pragma unroll
        for (int k = 0; k < 16; ++k) lo[k] = pool[k * kYStride + up];
        const double ha = 0.5 * fmax(shi, pool[16 * kYStride + up]);
        __syncthreads();                      // the y exchange has been read
        double H[10];
#pragma unroll
        for (int k = 0; k < 10; ++k) {
            H[k] = face_flux<1>(hi, lo, k, ha, im);
            pool[k * kYStride + ts] = H[k];
        }
        // this half writes the block's results and loads U_n meanwhile
        const int cols = nx - i0 < kCols ? nx - i0 : kCols, rows = ny - j0 < kRows ? ny - j0 : kRows;
        const size_t g0 = ((size_t)j0 * nx + i0) * 10, stride = (size_t)nx * 10;
        const double* Un = (A.a != 0.0 ? S.Un[sp] : Us) + g0;    // first stage: weight 0
        const unsigned o = tid < cols * 10 ? (unsigned)tid : 0u;
        double un[kRows];
#pragma unroll
        for (int jj = 0; jj < kRows; ++jj) un[jj] = (Un + (jj < rows ? jj : 0) * stride)[o];
        __syncthreads();                      // the y fluxes are stored
        const int dn = ty > 0 ? t - kCols : t;
#pragma unroll
        for (int k = 0; k < 10; ++k) H[k] = (H[k] - pool[k * kYStride + dn]) * A.idy;
        if (lane && ty >= 1 && ty <= kRows) {
            double* d = part + (ty - 1) * (kCols + 2) + tx + 1;
#pragma unroll
            for (int k = 0; k < 10; ++k) d[k * kXStride] = H[k];
        }
        __syncthreads();                      // the y differences are stored
        __syncthreads();                      // the results are stored
        if (tid < cols * 10) {
            double* Uo = S.Uo[sp] + g0;
            const bool first = A.a == 0.0;
#pragma unroll
            for (int jj = 0; jj < kRows; ++jj) {
                const double v = pool[jj * kCols * 10 + tid];
                if (jj < rows) (Uo + jj * stride)[(unsigned)tid] = first ? v : fma(A.b, v, A.a * un[jj]);
            }
        }
    }
}

// ------------------------------------------------------------------- 1V ----
// One SSP-RK3 step of the 1V fluid in one launch.  A block advances kLineTile
// cells: it holds them with six halo cells on each side (two per stage), runs
// the three stages in shared memory on a range that shrinks by two cells per
// side and stage, and writes its own cells to Uout, which must not be U unless
// one block covers the grid (another block reads U's halo).  The step is a
// chain of tiny dependent kernels otherwise: two launches per stage and the
// stage fields took 12 launches, about 3 us each whatever the grid.
// G.g set: the stage fields are the Poisson solves of the densities at t and
// t+1 and their mean, formed here; else they are read from E_t, E_t1, E_th.
struct LineFluid {
    const double* U;
    double* Uout;
    const double* mom_t;
    const double* mom_t1;
    const double* E_t;
    const double* E_t1;
    const double* E_th;
    const double* g;
    double dt, q, m, dx;
    int nx;
};
constexpr int kLineTile = 56;                 // + 8: the 64 cells whose fields the stages need
constexpr int kLineCells = kLineTile + 12;

__global__ void __launch_bounds__(256) line_rk3_kernel(LineFluid G) {
    __shared__ PoissonLds<2> P;
    __shared__ double cur[4][kLineCells], lo[4][kLineCells], hi[4][kLineCells], F[3][kLineCells];
    const int c = threadIdx.x;                // cell i0 - 6 + c
    const int i0 = blockIdx.x * kLineTile;
    const bool in = c < kLineCells;
    const int i = (int)((((long long)i0 - 6 + c) % G.nx + G.nx) % G.nx);
    double un[3] = {0.0, 0.0, 0.0}, qa = 0.0, qb = 0.0;
    if (in) {
#pragma unroll
        for (int k = 0; k < 3; ++k) un[k] = G.U[3ll * i + k];
        qa = G.mom_t[4ll * i + 3];
        qb = G.mom_t1[4ll * i + 3];
    }
    if (G.g) {
        const double* const src[2] = {G.mom_t, G.mom_t1};
        poisson_tile<2>(src, G.nx, G.g, i0 - 4, G.q, P);
    }
    double us[3] = {un[0], un[1], un[2]};
    const double m = G.m;
    auto spd = [m](const double* V) {
        const double u = V[1] / V[0], mn = m * V[0];
        const double p = fma(-u, mn * u, V[2]);
        return fabs(u) + sqrt(fmax(3.0 * p / mn, 0.0));
    };
#pragma unroll 1
    for (int s = 0; s < 3; ++s) {
        const int r = 2 * (s + 1);            // this stage updates cells [r, kLineCells - r)
        if (in) {
#pragma unroll
            for (int k = 0; k < 3; ++k) cur[k][c] = us[k];
            cur[3][c] = s == 0 ? qa : (s == 1 ? qb : 0.5 * qa + 0.5 * qb);
        }
        __syncthreads();
        if (c >= r - 1 && c < kLineCells - r + 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) cweno(cur[k][c - 1], cur[k][c], cur[k][c + 1], lo[k][c], hi[k][c]);
        }
        __syncthreads();
        if (c >= r - 1 && c < kLineCells - r) {          // face c + 1/2
            const double Um[4] = {hi[0][c], hi[1][c], hi[2][c], hi[3][c]};
            const double Up[4] = {lo[0][c + 1], lo[1][c + 1], lo[2][c + 1], lo[3][c + 1]};
            const double a = fmax(spd(Um), spd(Up));
            const double Fm[3] = {Um[1], Um[2] / m, Um[3]}, Fp[3] = {Up[1], Up[2] / m, Up[3]};
#pragma unroll
            for (int k = 0; k < 3; ++k) F[k][c] = 0.5 * (Fp[k] + Fm[k]) - 0.5 * a * (Up[k] - Um[k]);
        }
        __syncthreads();
        if (c >= r && c < kLineCells - r) {
            double e;
            if (G.g) {
                const double et = P.e[0][c - 2], et1 = P.e[1][c - 2];
                e = s == 0 ? et : (s == 1 ? et1 : 0.5 * et + 0.5 * et1);
            } else {
                e = (s == 0 ? G.E_t : (s == 1 ? G.E_t1 : G.E_th))[i];
            }
            const double a = s == 0 ? 0.0 : (s == 1 ? 0.75 : 1.0 / 3.0), b = s == 0 ? 1.0 : (s == 1 ? 0.25 : 2.0 / 3.0);
            const double f[3] = {0.0, (G.q / m) * us[0], 2.0 * G.q * us[1]};     // source: f e
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double v = fma(G.dt, fma(f[k], e, -((F[k][c] - F[k][c - 1]) / G.dx)), us[k]);
                us[k] = fma(b, v, a != 0.0 ? a * un[k] : 0.0);
            }
        }
        __syncthreads();
    }
    if (c >= 6 && c < 6 + kLineTile && i0 + c - 6 < G.nx) {
#pragma unroll
        for (int k = 0; k < 3; ++k) G.Uout[3ll * i + k] = us[k];
    }
}

__global__ void __launch_bounds__(256) copy_kernel(const double* __restrict__ a, double* __restrict__ b, long long n) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) b[i] = a[i];
}

// -------------------------------------------------------------- launchers --
// One SSP-RK3 step of ns species with the kinetic third moment (one launch per
// stage).  work: per species U1, U2 (10 doubles per cell each) at a stride of
// fluid_rk3_3v_doubles(nx, ny).
hipError_t launch_fluid_rk3_3v_set(int ns, double* const* U, const double* const* mom_t, const double* const* mom_t1,
                                   const double* E_t, const double* B_t, const double* E_t1, const double* B_t1,
                                   const double* E_th, const double* B_th, double dt, int nx, int ny, const double* q,
                                   const double* m, double dx, double dy, double* work, hipStream_t st, int per) {
    if (ns < 1 || ns > 2) return hipErrorInvalidValue;
    const double* E[3] = {E_t, E_t1, E_th};
    const double* B[3] = {B_t, B_t1, B_th};
    const double wa[3] = {1.0, 1.0, 0.5}, wb[3] = {0.0, 0.0, 0.5};
    for (int k = 0; k < 3; ++k) {
        FluidSet S{};
        for (int s = 0; s < ns; ++s) {
            rk3_buffers(S, s, k, U[s], work + (size_t)s * fluid_rk3_3v_doubles(nx, ny), (long long)nx * ny);
            S.QA[s] = k == 1 ? mom_t1[s] : mom_t[s];
            S.QB[s] = mom_t1[s];
            S.m[s] = m[s];
            S.q[s] = q[s];
        }
        const hipError_t e = launch_fluid_stage_3v_set(S, ns, kThirdFromF, k, wa[k], wb[k], E[k], B[k], dt, nx, ny, dx,
                                                       dy, st, per);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_fluid_stage_3v_set(const FluidSet& S, int ns, int third, int stage, double wa, double wb,
                                     const double* E, const double* B, double dt, int nx, int ny, double dx,
                                     double dy, hipStream_t st, int per) {
    if (ns < 1 || ns > 2 || stage < 0 || stage > 2) return hipErrorInvalidValue;
    const double a[3] = {0.0, 0.75, 1.0 / 3.0}, b[3] = {1.0, 0.25, 2.0 / 3.0};
    const int tx = (nx + kCols - 1) / kCols, ty = (ny + kRows - 1) / kRows;
    if ((long long)tx * ty * ns > 0x7fffffffll) return hipErrorInvalidValue;
    const FluidArgs A{nx, ny, 1.0 / dx, 1.0 / dy, a[stage], b[stage], dt, wa, wb, E, B, per, tx, ty};
    const dim3 grid((unsigned)((long long)tx * ty * ns)), blk(2 * kHalf);
    if (third == kThirdFromF)
        hipLaunchKernelGGL(fluid3_stage_kernel<kThirdKinetic>, grid, blk, 0, st, S, A);
    else if (third == kThirdGradient)
        hipLaunchKernelGGL(fluid3_stage_kernel<kThirdZero>, grid, blk, 0, st, S, A);
    else
        hipLaunchKernelGGL(fluid3_stage_kernel<kThirdNet>, grid, blk, 0, st, S, A);
    return hipGetLastError();
}

hipError_t launch_fluid_rk3_1v(double* U, double* Uout, const double* mom_t, const double* mom_t1, const double* E_t,
                               const double* E_t1, const double* E_th, const double* g, double dt, int nx, double q,
                               double m, double dx, double* work, hipStream_t st) {
    const int blocks = (nx + kLineTile - 1) / kLineTile;
    double* to = (Uout != U || blocks == 1) ? Uout : work;
    LineFluid G{U, to, mom_t, mom_t1, E_t, E_t1, E_th, g, dt, q, m, dx, nx};
    hipLaunchKernelGGL(line_rk3_kernel, dim3(blocks), dim3(256), 0, st, G);
    if (to != Uout)
        hipLaunchKernelGGL(copy_kernel, dim3((3 * nx + 255) / 256), dim3(256), 0, st, work, Uout, 3ll * nx);
    return hipGetLastError();
}

}  // namespace vl
