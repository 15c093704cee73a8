// PFC advection sweeps for gfx950: x (periodic), y (reflecting walls, pencil
// pairs +v_y / -v_y), v in 1V (zero-flux) and the five-sweep 3V velocity
// operator (zero-flux), plus the array maximum that bounds the limiter.
//
// Scheme: positive and flux-conservative semi-Lagrangian sweep (Sec. 2.1 of
// arXiv 2109.06743, which uses the PFC scheme of Filbet, Sonnendruecker and
// Bertrand).  For a uniform displacement s = K + a (K = floor, s >= 0) the
// flux-form update telescopes to
//     f'_i = f_{i-K} + phi(i-K-1) - phi(i-K),
// phi(j) the limited partial flux of cell j (pfc_phi).  Negative shifts run
// the same formula on the mirrored pencil.  Integer shifts give a = 0 and
// therefore an exact (bitwise) shift.
#include <climits>

#include "vl_internal.h"

namespace vl {

// ---------------------------------------------------------------------------
// x sweep: layout [rows][nx][Nv]; each thread owns one velocity index v of one
// row and CX consecutive output cells; lanes run over contiguous v, so every
// load and store of a wave is one contiguous 256-byte (FP32) segment.  The
// thread keeps a window of CX+3 inputs in registers, ordered upwind to
// downwind, so both signs of the shift run the same straight-line code.
// Offsets within a row are 32-bit (nx * Nv < 2^31 is checked on the host) and
// advance by one row per element; only windows that cross the periodic seam
// take the wrapping path.
template <class T, int CX, bool kFold>
__global__ void __launch_bounds__(256)
pfc_x_kernel(const T* __restrict__ fin, T* __restrict__ fout, int nx, int Nv, float inv_inner, double vx_lo,
             double dvx, double tau_dx, MaxRef finf_r, typename Bits<T>::U* __restrict__ max_out) {
    // work index = (v block fastest, then x chunk, then row), XCD-contiguous
    const unsigned nvb = (Nv + 255) / 256, nch = (nx + CX - 1) / CX;
    const unsigned w = xcd_work_index(blockIdx.x, gridDim.x);
    const int v = (int)(w % nvb) * 256 + threadIdx.x;
    const int c0 = (int)((w / nvb) % nch) * CX;
    const size_t rowoff = (size_t)(w / (nvb * nch)) * nx * Nv;
    const T* __restrict__ src = fin + rowoff;
    T* __restrict__ dst = fout + rowoff;
    const T F2 = T(2) * max_of<T, kFold>(finf_r);
    T mx = T(0);
    if (v < Nv) {
        const int ivx = row_of(v, inv_inner);
        const double s = (vx_lo + (ivx + 0.5) * dvx) * tau_dx;
        const bool pos = s >= 0.0;
        const Shift<T> sh(fabs(s));
        const int K = sh.K < nx ? (int)sh.K : (int)(sh.K % nx);
        int idx = pos ? (c0 - K - 2) : (c0 + K + CX + 1);
        while (idx < 0) idx += nx;
        while (idx >= nx) idx -= nx;
        const int step = pos ? 1 : -1;
        const unsigned dstep = pos ? (unsigned)Nv : (unsigned)(-Nv);
        unsigned off = (unsigned)idx * (unsigned)Nv + (unsigned)v;
        T W[CX + 3];
        const bool wraps = pos ? (idx + CX + 2 >= nx) : (idx - CX - 2 < 0);
        if (!wraps) {
#pragma unroll
            for (int w = 0; w < CX + 3; ++w) {
                W[w] = src[off];
                off += dstep;
            }
        } else {
            const unsigned span = (unsigned)nx * (unsigned)Nv;
#pragma unroll
            for (int w = 0; w < CX + 3; ++w) {
                W[w] = src[off];
                idx += step;
                off += dstep;
                if (idx == nx) {
                    idx = 0;
                    off -= span;
                } else if (idx < 0) {
                    idx = nx - 1;
                    off += span;
                }
            }
        }
        T o[CX];
        T D = W[2] - W[1];
        T phi_prev = pfc_phi_d(W[1], W[1] - W[0], D, sh.a, sh.ac1, sh.ac2, F2);
#pragma unroll
        for (int r = 0; r < CX; ++r) {
            const T Dn = W[r + 3] - W[r + 2];
            const T phi_next = pfc_phi_d(W[r + 2], D, Dn, sh.a, sh.ac1, sh.ac2, F2);
            o[r] = fmax(W[r + 2] + phi_prev - phi_next, T(0));
            phi_prev = phi_next;
            D = Dn;
        }
        unsigned ooff = (unsigned)(pos ? c0 : c0 + CX - 1) * (unsigned)Nv + (unsigned)v;
        if (c0 + CX <= nx) {
#pragma unroll
            for (int r = 0; r < CX; ++r) {
                dst[ooff] = o[r];
                mx = fmax(mx, o[r]);
                ooff += dstep;
            }
        } else {
#pragma unroll
            for (int r = 0; r < CX; ++r) {
                if ((pos ? c0 + r : c0 + CX - 1 - r) < nx) {
                    dst[ooff] = o[r];
                    mx = fmax(mx, o[r]);
                }
                ooff += dstep;
            }
        }
    }
    if (max_out) block_max_part(mx, max_out);
}

// Partial flux a w + cA A + cB B of a cell with value w and neighbour
// differences Dm (below) and Dp (above), F2 = 2 f_inf: the limited slopes are
// A = med3(Dp, -r2, 2w) and B = med3(Dm, -2w, r2) with r2 = F2 - 2w taken
// without its clamp at zero (see the cubic velocity sweeps below).
template <class T>
__device__ __forceinline__ T sub_cell_flux(T w, T Dm, T Dp, T a, T cA, T cB, T F2) {
    const T x2 = w + w;
    const T r2 = F2 - x2;
    const T A = med3(Dp, -r2, x2);
    const T B = med3(Dm, -x2, r2);
    return fma(cA, A, fma(cB, B, a * w));
}

// ---------------------------------------------------------------------------
// Fused X(tau) for 2X3V: the x sweep and then the y sweep with one f_inf, in
// one pass over f.
//
// Work item: one wave = 64 consecutive velocity indices of the block (a
// "chunk"; the block of a cell is contiguous, so a wave's access to one cell
// is a 256-byte run -- whole 128-byte lines wherever the block size is a
// multiple of 32 elements), C adjacent x cells (a strip) and a segment of S
// rows.  Every lane owns one velocity v and writes only v.  All lanes walk
// the rows upward together, so each step reads the same row in every lane
// and the wave reads whole lines of it: a lane whose v_y is negative walks
// against its flow and emits each output K_y + 1 rows after the upward
// lanes (its output at row r depends on the x-swept rows r+K_y-1 .. r+K_y+2,
// which it holds by then).
//
// y boundary, with virtual rows q outside [0, ny): periodic: row q mod ny of
// v itself.  Reflecting walls: the pencil of v continues beyond a wall with
// the pencil of its mirror velocity v' (v_y -> -v_y) read backwards, i.e.
// q mod 2ny = q' < ny is row q' of v and q' >= ny is row 2ny-1-q' of v'.
// Both velocities of a mirror pair take the shift of the positive one, so
// the flux through a wall that the lane of v sends out and the flux the lane
// of v' takes in are computed from the same values in the same order: the
// wall exchange conserves mass exactly.
//
// For each row the x sweep of the C cells runs on the fly (a window of C+3
// inputs in registers, three rows of loads in flight while one is
// computed) and feeds the y update, so the x-swept array never reaches
// memory.  A load is a wave-uniform row base plus a per-lane 32-bit byte
// offset; the stores of one step (rows i-2-Kmax .. i-1+Kmax across the wave)
// are a wave-uniform base plus per-lane 32-bit offsets where those rows span
// less than 4 GiB (WIDE = false), else a per-lane 64-bit address.
// Work order: chunk fastest, then strip, then segment, so the waves in
// flight cover whole rows and neighbouring strips (x halos) together.
struct XYArgs {
    int nx, ny, Nv, nvy, nvz, S, nchunks, nst, nseg, per;
    int pad;              // entries of max_out; those beyond the grid's are set to 0
    float inv_nvz, inv_nvyz;
    double vx_lo, dvx, tau_dx, vy_lo, dvy, tau_dy;
};

template <class T, int C, bool WIDE, bool kFold>
__global__ void __launch_bounds__(256)
pfc_xy_kernel(const T* __restrict__ fin, T* __restrict__ fout, XYArgs A, MaxRef finf_r,
              typename Bits<T>::U* __restrict__ max_out) {
    const unsigned gw = xcd_work_index(blockIdx.x, gridDim.x) * 4u + (threadIdx.x >> 6);
    const int lane = threadIdx.x & (kWave - 1);
    const unsigned chunk = gw % (unsigned)A.nchunks;
    const unsigned rest = gw / (unsigned)A.nchunks;
    const int c0 = (int)(rest % (unsigned)A.nst) * C;
    const unsigned seg = rest / (unsigned)A.nst;
    const T F2 = T(2) * max_of<T, kFold>(finf_r);
    T mx = T(0);
    if (seg < (unsigned)A.nseg) {                    // wave-uniform
        const int nx = A.nx, ny = A.ny, Nv = A.Nv;
        const int vl = (int)chunk * kWave + lane;
        const bool active = vl < Nv;
        const int v = active ? vl : Nv - 1;          // idle lanes walk a real pencil and store nothing
        const int ivx = row_of(v, A.inv_nvyz);
        const int jy = row_of(v, A.inv_nvz) - ivx * A.nvy;
        const int jm = A.nvy - 1 - jy;
        const bool up = jy >= jm;                    // v_y >= 0 (an odd grid's middle cell does not move)
        // y: both members of a mirror pair move by the shift of the positive one
        const double syd = (jy == jm) ? 0.0 : (A.vy_lo + ((up ? jy : jm) + 0.5) * A.dvy) * A.tau_dy;
        const ShiftT<T> shy(syd);
        const int L = A.per ? ny : 2 * ny;
        const int Ky = shy.K < L ? shy.K : shy.K % L;
        int Kmax = Ky;
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) Kmax = max(Kmax, __shfl_xor(Kmax, o, kWave));
        Kmax = __builtin_amdgcn_readfirstlane(Kmax);
        // x: uniform shift along the row
        const double sxd = (A.vx_lo + (ivx + 0.5) * A.dvx) * A.tau_dx;
        const bool posx = sxd >= 0.0;
        const Shift<T> shx(fabs(sxd));
        const int Kx = shx.K < nx ? (int)shx.K : (int)(shx.K % nx);
        int col = posx ? c0 - Kx - 2 : c0 + Kx + C + 1;  // first (upwind) column of the x window
        while (col < 0) col += nx;
        while (col >= nx) col -= nx;
        unsigned boff[C + 3];
#pragma unroll
        for (int w = 0; w < C + 3; ++w) {
            boff[w] = ((unsigned)col * (unsigned)Nv + (unsigned)v) * (unsigned)sizeof(T);
            col += posx ? 1 : -1;
            if (col == nx) col = 0;
            if (col < 0) col = nx - 1;
        }
        const unsigned dmir = (unsigned)((jm - jy) * A.nvz) * (unsigned)sizeof(T);   // v' - v (mod 2^32)
        const size_t rowbytes = (size_t)nx * Nv * sizeof(T);
        // output rows of the segment and the steps that produce them
        const int r0 = (int)seg * A.S;
        const int r1 = min(r0 + A.S, ny);
        const int ib = r0 + 1 - Kmax, ie = r1 + 1 + Kmax;
        const int dr = up ? Ky - 1 : -2 - Ky;        // output row = step + dr
        const int ilo = active ? r0 - dr : INT_MAX, ihi = r1 - dr;
        const int drmin = -2 - Kmax;
        unsigned soff[C];
        bool colok[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int oc = posx ? c0 + c : c0 + C - 1 - c;   // the x outputs run upwind to downwind
            colok[c] = oc < nx;
            const unsigned within = ((unsigned)oc * (unsigned)Nv + (unsigned)v) * (unsigned)sizeof(T);
            soff[c] = WIDE ? within : (unsigned)(dr - drmin) * (unsigned)rowbytes + within;
        }
        const bool full = c0 + C <= nx;
        // virtual row q -> (row, mirror?): wave-uniform
        auto load = [&](int q, T (&W)[C + 3]) {
            int row = q;
            bool mir = false;
            if ((unsigned)q >= (unsigned)ny) {
                row = q % L;
                if (row < 0) row += L;
                if (!A.per && row >= ny) {
                    mir = true;
                    row = L - 1 - row;
                }
            }
            const char* base = reinterpret_cast<const char*>(fin) + (size_t)row * rowbytes;
            if (!mir) {
#pragma unroll
                for (int w = 0; w < C + 3; ++w) W[w] = *reinterpret_cast<const T*>(base + boff[w]);
            } else {
#pragma unroll
                for (int w = 0; w < C + 3; ++w) W[w] = *reinterpret_cast<const T*>(base + (boff[w] + dmir));
            }
        };
        // partial flux without the clamp of r2 at zero: every sweep's input
        // lies in [0, f_inf] up to rounding (as in the velocity sweeps)
        auto xsweep = [&](const T (&W)[C + 3], T (&P)[C]) {
            T D = W[2] - W[1];
            T phi_prev = sub_cell_flux(W[1], W[1] - W[0], D, shx.a, shx.ac1, shx.ac2, F2);
#pragma unroll
            for (int r = 0; r < C; ++r) {
                const T Dn = W[r + 3] - W[r + 2];
                const T phi_next = sub_cell_flux(W[r + 2], D, Dn, shx.a, shx.ac1, shx.ac2, F2);
                P[r] = fmax(W[r + 2] + phi_prev - phi_next, T(0));
                phi_prev = phi_next;
                D = Dn;
            }
        };
        // y state per column: P1 = P(i-1), P2 = P(i-2) and ph = the flux of
        // cell i-2 in the lane's direction of motion (up: through its upper
        // face, from P(i-3), P(i-2), P(i-1); down: through its lower face)
        T P1[C], P2[C], ph[C];
        {
            T Wa[C + 3], Pa[C];
            load(ib - 3, Wa);
            xsweep(Wa, Pa);
            load(ib - 2, Wa);
            xsweep(Wa, P2);
            load(ib - 1, Wa);
            xsweep(Wa, P1);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T d1 = P2[c] - Pa[c], d0 = P1[c] - P2[c];
                ph[c] = sub_cell_flux(P2[c], up ? d1 : -d0, up ? d0 : -d1, shy.a, shy.ac1, shy.ac2, F2);
            }
        }
        // step i: x-sweep row i (window Wc), the flux of cell i-1, the
        // output of cell i-1 (up, stored at row i-1+Ky) or i-2 (down, at row
        // i-2-Ky); the window of row i+3 is loaded into Wn meanwhile
        auto step = [&](int i, const T (&Wc)[C + 3], T (&Wn)[C + 3]) {
            if (i + 3 <= ie) load(i + 3, Wn);
            T P0[C];
            xsweep(Wc, P0);
            T o[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T d1 = P1[c] - P2[c], d0 = P0[c] - P1[c];
                const T phn = sub_cell_flux(P1[c], up ? d1 : -d0, up ? d0 : -d1, shy.a, shy.ac1, shy.ac2, F2);
                const T base = up ? P1[c] : P2[c];
                const T fin_ = up ? ph[c] : phn;
                const T fout_ = up ? phn : ph[c];
                o[c] = fmax(base + fin_ - fout_, T(0));
                ph[c] = phn;
                P2[c] = P1[c];
                P1[c] = P0[c];
            }
            if (i >= ilo && i < ihi) {
                char* ob = WIDE ? reinterpret_cast<char*>(fout) + (size_t)(i + dr) * rowbytes
                                : reinterpret_cast<char*>(fout) + (long long)(i + drmin) * (long long)rowbytes;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if (full || colok[c]) {
                        *reinterpret_cast<T*>(ob + soff[c]) = o[c];
                        mx = max_nonneg(mx, o[c], F2);
                    }
                }
            }
        };
        T W0[C + 3], W1[C + 3], W2[C + 3], W3[C + 3];
        load(ib, W0);
        if (ib + 1 <= ie) load(ib + 1, W1);
        if (ib + 2 <= ie) load(ib + 2, W2);
        int i = ib;
        for (; i + 3 <= ie; i += 4) {                 // four rows: the windows rotate
            step(i, W0, W3);
            step(i + 1, W1, W0);
            step(i + 2, W2, W1);
            step(i + 3, W3, W2);
        }
        if (i <= ie) step(i, W0, W3);
        if (i + 1 <= ie) step(i + 1, W1, W0);
        if (i + 2 <= ie) step(i + 2, W2, W1);
    }
    if (max_out) {
        block_max_part(mx, max_out);
        if (blockIdx.x == 0)
            for (int k = (int)(gridDim.x + threadIdx.x); k < A.pad; k += 256) max_out[k] = 0;
    }
}

// ---------------------------------------------------------------------------
// 3V velocity operator by the backsubstitution split.  The step's velocity
// map under the cell's uniform E, B is the implicit-midpoint (Boris) map
// v -> R v + c, R = I + [s](I + [t]) with t = (q tau/2m) B, s = 2t/(1+t.t)
// and [a]v = v x a, c = (I + R)(q tau/2m) E.  Row by row it factors into an
// x-, a y- and a z-map that each change one component from the components
// already updated (x' = a x + b y + e z + cx; y' = d x' + g y + h z + cy;
// z' = k x' + l y' + n z + cz).  Each map is affine along its pencils: the
// stretch is the cell's (a, g or n), the shift linear in the pencil's
// transverse cell-centre velocities.  Coefficients in FP64.
__device__ __forceinline__ void backsub_coeffs(const double* EB, double qm, double tau, double* C) {
    const double h = 0.5 * qm * tau;
    const double t[3] = {h * EB[3], h * EB[4], h * EB[5]};
    const double k = 2.0 / (1.0 + t[0] * t[0] + t[1] * t[1] + t[2] * t[2]);
    const double s[3] = {k * t[0], k * t[1], k * t[2]};
    // [a] as a matrix: [a]v = v x a
    auto X = [](const double* a, double (&M)[3][3]) {
        M[0][0] = 0.0;   M[0][1] = a[2];  M[0][2] = -a[1];
        M[1][0] = -a[2]; M[1][1] = 0.0;   M[1][2] = a[0];
        M[2][0] = a[1];  M[2][1] = -a[0]; M[2][2] = 0.0;
    };
    double S[3][3], T[3][3], R[3][3];
    X(s, S);
    X(t, T);
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double acc = S[i][j] + (i == j ? 1.0 : 0.0);
            for (int l = 0; l < 3; ++l) acc += S[i][l] * T[l][j];
            R[i][j] = acc;
        }
    double c[3];
    for (int i = 0; i < 3; ++i) c[i] = h * (EB[i] + R[i][0] * EB[0] + R[i][1] * EB[1] + R[i][2] * EB[2]);
    const double a = R[0][0], b = R[0][1], e = R[0][2];
    const double d = R[1][0] / a;
    const double g = R[1][1] - d * b, hh = R[1][2] - d * e;
    const double det = R[0][0] * R[1][1] - R[0][1] * R[1][0];
    const double kk = (R[2][0] * R[1][1] - R[2][1] * R[1][0]) / det;
    const double l = (R[0][0] * R[2][1] - R[0][1] * R[2][0]) / det;
    const double n = R[2][2] - kk * R[0][2] - l * R[1][2];
    C[0] = a;  C[1] = b;  C[2] = e;  C[3] = c[0];
    C[4] = d;  C[5] = g;  C[6] = hh; C[7] = c[1] - d * c[0];
    C[8] = kk; C[9] = l;  C[10] = n; C[11] = c[2] - kk * c[0] - l * c[1];
}

// One affine sweep along an axis: the content at cell coordinate xi (cell j =
// [j, j+1]) moves to alpha xi + sigma, so face i has its foot at
// F_i = (i - sigma)/alpha = i + delta_i, delta_i = i (1/alpha - 1) - sigma/alpha.
// The wall faces carry no flux.
//
// Every foot within a cell of its face (|delta_i| < 1, the common case; delta
// is linear in i, so the end faces decide): the flux through face i is
//   delta < 0:  phi(i-1, a),  a = -delta, the mass of the cell below within a
//               of its upper face: a (w + c1 A + c2 B),
//   delta >= 0: minus the mass of the cell above within a = delta of its lower
//               face, the mirrored flux: -a (w - c1 B - c2 A),
// with A, B the limited slopes of that cell (sub_cell_flux; the bound on the
// values is max(f_inf, w), as a sweep with alpha < 1 raises them), so both are
// -delta w + a c1 U + a c2 V with (U, V) = (A, B) of the cell below or (B, A) of
// the cell above: a select of three values per face.
template <class T, int N>
__device__ __forceinline__ void affine_exact(T (&g)[N], T d0, T d1, T F2) {
    T w0 = g[0], A0, B0;
    T Dp = g[1] - g[0];
    {
        const T x2 = w0 + w0, r2 = fmax(F2 - x2, T(0));
        A0 = med3(Dp, -r2, x2);
        B0 = med3(w0, -x2, r2);              // zero ghost below
    }
    T Fprev = T(0);
#pragma unroll
    for (int m = 0; m < N - 1; ++m) {        // face m + 1, between cells m and m + 1
        const T w1 = g[m + 1];
        const T Dm1 = Dp, Dp1 = (m + 2 < N ? g[m + 2 < N ? m + 2 : m] : T(0)) - w1;
        const T x2 = w1 + w1, r2 = fmax(F2 - x2, T(0));
        const T A1 = med3(Dp1, -r2, x2), B1 = med3(Dm1, -x2, r2);
        const T delta = fma((T)(m + 1), d1, d0);
        const bool up = delta < T(0);
        const T aa = fabs(delta);
        const T t = (aa - aa * aa) * T(1.0 / 6.0);
        const T ac1 = fma(-t, aa, t + t), ac2 = fma(t, aa, t);
        const T w = up ? w0 : w1, U = up ? A0 : B1, V = up ? B0 : A1;
        const T F = fma(ac1, U, fma(ac2, V, -delta * w));
        g[m] = fmax(w0 + Fprev - F, T(0));
        Fprev = F;
        w0 = w1;
        A0 = A1;
        B0 = B1;
        Dp = Dp1;
    }
    g[N - 1] = fmax(w0 + Fprev, T(0));
}

// The general case, one pencil in shared memory: the feet clamped to the box
// [0, N] (F_0 = 0, F_N = N); F = j + t (0 <= t < 1) splits a foot, and
// R = phi(j, 1 - t) is the mass of cell j above it (phi the limited partial flux;
// R = f_j exactly at t = 0, 0 beyond the box).  Output cell i holds the mass
// between its two feet:
//   j_{i+1} == j_i:  R_i - R_{i+1}
//   else:            R_i + f_{j_i+1} + ... + f_{j_{i+1}-1} + (f_{j_{i+1}} - R_{i+1}),
// so whole-cell moves are exact and the pencil's mass telescopes.  A foot's
// three cells are read at indices clamped to the pencil and set to zero beyond
// it: with a branch around each read, and the length a run-time number, a face
// took 150 instructions instead of about 50, and a wave that holds pencils of
// both kinds runs this after affine_exact.
template <class T, int N>
__device__ __attribute__((noinline)) void affine_far(LdsPtr<T> pc, int stride, T ia, T ib, T F2) {
    auto at = [&](int k) -> T { return pc[__umul24((unsigned)k, (unsigned)stride)]; };
    T out[N];
    int jp = 0;
    T Rp = pc[0];                                   // face 0: F = 0
#pragma unroll
    for (int i = 0; i < N; ++i) {
        int j = N;
        T R = T(0), f0 = T(0);                      // face N: F = N
        if (i + 1 < N) {
            const T F = fmin(fmax(fma((T)(i + 1), ia, ib), T(0)), (T)N);
            const T fj = floor(F);
            j = (int)fj;
            const T t = F - fj;
            const T m0 = at(j < N ? j : N - 1), mm = at(j > 0 ? j - 1 : 0), mp = at(j + 1 < N ? j + 1 : N - 1);
            f0 = j < N ? m0 : T(0);
            const T fm = j > 0 ? mm : T(0), fp = j + 1 < N ? mp : T(0);
            const T c1 = fma(t, t, t) * T(1.0 / 6.0), c2 = (t + t - t * t) * T(1.0 / 6.0);
            const T f2 = f0 + f0, r2 = fmax(F2 - f2, T(0));
            R = (T(1) - t) * fma(c2, med3(f0 - fm, -f2, r2), fma(c1, med3(fp - f0, -r2, f2), f0));
        }
        T acc = Rp;
#pragma unroll 1
        for (int m = jp + 1; m < j; ++m) acc += at(m);
        out[i] = fmax(j == jp ? Rp - R : acc + (f0 - R), T(0));
        asm volatile("" : "+v"(out[i]));            // formed here: moved to the stores, it holds seven registers a face
        jp = j;
        Rp = R;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) pc[i * stride] = out[i];
}

// One pencil of N cells (kIn: read from global memory) into shared memory.
template <class T, int N, bool kIn>
__device__ __forceinline__ void affine_pencil(const T* __restrict__ src, unsigned plane, T* pc, int stride, double ia,
                                              double sa, T finf) {
    T g[N];
    if constexpr (kIn) {
#pragma unroll
        for (int m = 0; m < N; ++m) g[m] = src[(unsigned)m * plane];
    } else {
#pragma unroll
        for (int m = 0; m < N; ++m) g[m] = pc[m * stride];
    }
    const T d1 = (T)(ia - 1.0), d0 = (T)(-sa);
    const T first = d0 + d1, last = fma((T)(N - 1), d1, d0);
    if (fabs(first) < T(1) && fabs(last) < T(1)) {
        affine_exact<T, N>(g, d0, d1, T(2) * finf);
#pragma unroll
        for (int m = 0; m < N; ++m) pc[m * stride] = g[m];
    } else {
        if constexpr (kIn) {
#pragma unroll
            for (int m = 0; m < N; ++m) pc[m * stride] = g[m];
        }
        affine_far<T, N>(lds_ptr(pc), stride, (T)ia, (T)(-sa), T(2) * finf);
    }
}

// One sweep of the cell's block.  C: the twelve coefficients of the factored
// map, then the reciprocals of its three stretches.
template <class T, bool kIn, int NEXACT, int LMAX>
__device__ __forceinline__ void sweep_affine(const T* __restrict__ src, T* blk, int dd, const double* C,
                                             const V3Params& P, T finf) {
    const int pz = P.nvz | 1;
    const int n = dd == 0 ? P.nvx : (dd == 1 ? P.nvy : P.nvz);
    const int npen = dd == 0 ? P.nvy * P.nvz : (dd == 1 ? P.nvx * P.nvz : P.nvx * P.nvy);
    const int n2 = dd == 2 ? P.nvy : P.nvz;
    const float inv_n2 = dd == 2 ? P.inv_nvy : P.inv_nvz;
    const double alpha = C[dd == 0 ? 0 : (dd == 1 ? 5 : 10)], ia = C[12 + dd];
    const double k1 = C[dd == 0 ? 1 : (dd == 1 ? 4 : 8)], k2 = C[dd == 0 ? 2 : (dd == 1 ? 6 : 9)],
                 k3 = C[dd == 0 ? 3 : (dd == 1 ? 7 : 11)];
    const int t1 = dd == 0 ? 1 : 0, t2 = dd == 2 ? 1 : 2;       // transverse axes
    // sigma = ((alpha - 1) lo + k1 v1 + k2 v2 + k3) / dv for v -> alpha v + ...
    const double s0 = (alpha - 1.0) * P.lo[dd] + k3;
    for (int pen = threadIdx.x; pen < npen; pen += blockDim.x) {
        const int i1 = row_of(pen, inv_n2), i2 = pen - i1 * n2;
        const int base = dd == 0 ? i1 * pz + i2 : (dd == 1 ? i1 * P.nvy * pz + i2 : (i1 * P.nvy + i2) * pz);
        const int stride = dd == 0 ? P.nvy * pz : (dd == 1 ? pz : 1);
        const double v1 = P.lo[t1] + (i1 + 0.5) * P.dv[t1], v2 = P.lo[t2] + (i2 + 0.5) * P.dv[t2];
        const double sa = (s0 + k1 * v1 + k2 * v2) * P.inv_dv[dd] * ia;      // sigma / alpha
        const unsigned plane = (unsigned)(P.nvy * P.nvz);
        if constexpr (NEXACT > 0) {
            affine_pencil<T, NEXACT, kIn>(src + pen, plane, blk + base, stride, ia, sa, finf);
        } else {
#define VL_LEN(N)                                                                                 \
    case N:                                                                                       \
        if constexpr (N <= LMAX) affine_pencil<T, N, kIn>(src + pen, plane, blk + base, stride, ia, sa, finf); \
        break;
            VL_LENGTHS(n)
#undef VL_LEN
        }
    }
}

// One block per cell, the block of f in shared memory, one pencil at a time per
// thread in registers; the first sweep's pencils come straight from global
// memory.  Bound by issue: a face costs about 25 instructions, three sweeps 75 a
// value, and the six selects and two clamps of the flux cannot use the packed or
// matrix units.  32768 cells of 12^3 FP32: 386 us when every face took its flux
// from the values around its foot in shared memory (a gather of three per face,
// behind an index computed from the foot), now 148; 5000 cells of 20x16x24
// FP32 371 -> 211 and 8192 of 16^3 FP64 358 -> 235 with the maximum of f taken
// first, 640 of 34^3 FP32 279 -> 162.  Six waves per SIMD (80 registers, spills)
// instead of four: 160.
//
// NEXACT: cube edge, or 0 for any axes of 2 to LMAX cells (code for each exact
// length, chosen by a switch).  LMAX 32 takes 255 registers in FP32, two waves
// a SIMD, because of the longest pencils; the cubes and grids of short axes have
// code of their own, which takes 79 to 117: 8^3 256x128 cells FP32 51 us against
// 56, 12^3 200x100 104 against 150, 16^3 232 against 334 (FP64 79, 198, 452
// against 80, 245, 536), 4^3 300x200 with axes up to 8 53 against 124.  Holding
// LMAX 32 to 128 registers spills: 20x16x24 100x50 383 against 175.
template <class T, int NEXACT, int LMAX, int NTH, bool kFold>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(LMAX <= 8 ? (sizeof(T) == 4 ? 6 : 4) : 1)))
pfc_v3b_kernel(const T* fin, T* fout, const double* __restrict__ E, const double* __restrict__ B,
               V3Params P, MaxRef finf_r, typename Bits<T>::U* __restrict__ max_out) {
    extern __shared__ unsigned char smem_raw[];
    T* blk = reinterpret_cast<T*>(smem_raw);
    __shared__ double Cs[15];
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const int nv = P.nvx * P.nvy * P.nvz;
    const int pz = P.nvz | 1;
    const T finf = max_of<T, kFold>(finf_r);
    if (threadIdx.x == 0) {
        double EB[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            EB[k] = E[cell * 3 + k];
            EB[3 + k] = B ? B[cell * 3 + k] : 0.0;
        }
        backsub_coeffs(EB, P.qm, P.tau, Cs);
        Cs[12] = 1.0 / Cs[0];
        Cs[13] = 1.0 / Cs[5];
        Cs[14] = 1.0 / Cs[10];
    }
    __syncthreads();
    const T* src = fin + cell * nv;
    sweep_affine<T, true, NEXACT, LMAX>(src, blk, 0, Cs, P, finf);
    __syncthreads();
#pragma unroll 1
    for (int d = 1; d < 3; ++d) {
        sweep_affine<T, false, NEXACT, LMAX>(src, blk, d, Cs, P, finf);
        __syncthreads();
    }
    T* dst = fout + cell * nv;
    T mx = T(0);
    for (int e = threadIdx.x; e < nv; e += blockDim.x) {
        const T o = blk[e + row_of(e, P.inv_nvz) * (pz - P.nvz)];
        dst[e] = o;
        mx = fmax(mx, o);
    }
    if (max_out) block_max_part(mx, max_out);
}

// ---------------------------------------------------------------------------
// Zero-flux sweep of one pencil held in shared memory, in upwind-to-downwind
// order g[0..n-1] with two zero ghosts on each side (index k lives at g[k+2]).
// With h_k = g_k + phi(k-1) - phi(k) (h_n = phi(n-1)), the output at position
// p is 0 for p < K, h_{p-K} for K <= p < n-1, and the wall cell n-1 keeps all
// the mass that would have crossed it: sum_{k >= n-1-K} h_k.
template <class T>
__device__ __forceinline__ T zeroflux_out(const T* g, int n, int p, long long K, const Shift<T>& sh, T finf) {
    if (p < n - 1) {
        if ((long long)p < K) return T(0);
        const int k = p - (int)K;
        const T pm = pfc_phi(g[k], g[k + 1], g[k + 2], sh.a, sh.c1, sh.c2, finf);   // phi(k-1)
        const T p0 = pfc_phi(g[k + 1], g[k + 2], g[k + 3], sh.a, sh.c1, sh.c2, finf); // phi(k)
        return fmax(g[k + 2] + pm - p0, T(0));
    }
    long long k0 = (long long)(n - 1) - K;
    if (k0 < 0) k0 = 0;
    T acc = T(0);
    T pm = pfc_phi(g[k0], g[k0 + 1], g[k0 + 2], sh.a, sh.c1, sh.c2, finf);
    for (int k = (int)k0; k <= n; ++k) {
        const T p0 = pfc_phi(g[k + 1], g[k + 2], g[k + 3], sh.a, sh.c1, sh.c2, finf);
        acc += g[k + 2] + pm - p0;
        pm = p0;
    }
    return fmax(acc, T(0));
}

// 1V velocity sweep: one block per spatial cell, the pencil staged in shared
// memory (nv + 4 values).  s = (q/m) E_i tau / dv.  In place is allowed.  E
// from S.E, or (S.g set) from the densities of the moments S.mom [nx][4] by
// the Poisson convolution (see poisson_tile), stored to S.E as well: the
// solve costs each block nx multiply-adds and the step two launches less.
struct LineField {
    double* E;
    const double* mom;
    const double* g;
    double q;
};
template <class T, bool kFold>
__global__ void __launch_bounds__(256)
pfc_v1_kernel(const T* fin, T* fout, int nx, int nv, LineField S, double qm_tau_dv,
              MaxRef finf_r, typename Bits<T>::U* __restrict__ max_out) {
    extern __shared__ unsigned char smem_raw[];
    __shared__ double red[4];
    T* g = reinterpret_cast<T*>(smem_raw);
    const int ix = blockIdx.x;
    double e;
    if (S.g) {
        const double own = S.mom[4ll * ix];
        double acc[1] = {0.0};
        for (int j = threadIdx.x; j < nx; j += blockDim.x)
            acc[0] = fma(S.mom[4ll * j] - own, S.g[ix >= j ? ix - j : ix - j + nx], acc[0]);
        block_sum<1>(acc, red);
        e = S.q * acc[0];
        if (threadIdx.x == 0) S.E[ix] = e;
    } else {
        e = S.E[ix];
    }
    const double s = qm_tau_dv * e;
    const bool pos = s >= 0.0;
    const Shift<T> sh(fabs(s));
    const T finf = max_of<T, kFold>(finf_r);
    const T* src = fin + (long long)ix * nv;
    T* dst = fout + (long long)ix * nv;
    for (int k = threadIdx.x; k < nv + 4; k += blockDim.x) {
        const int j = k - 2;
        g[k] = (j >= 0 && j < nv) ? src[pos ? j : nv - 1 - j] : T(0);
    }
    __syncthreads();
    T mx = T(0);
    for (int p = threadIdx.x; p < nv; p += blockDim.x) {
        const T o = zeroflux_out(g, nv, p, sh.K, sh, finf);
        dst[pos ? p : nv - 1 - p] = o;
        mx = fmax(mx, o);
    }
    if (max_out) block_max_part(mx, max_out);
}

// ---------------------------------------------------------------------------
// 3V velocity operator V(tau) on any velocity grid (axes of 2 to 32 cells):
// one block per spatial cell, the velocity block in shared memory with rows
// along v_z padded to an odd length, so a wave reading pencils along any of the
// three axes hits distinct banks.  The five sweeps are vx(tau/2) vy(tau/2)
// vz(tau) vy(tau/2) vx(tau/2), each a uniform shift by
// (q/m)(E_d + (v x B)_d) at the pencil's transverse velocities; a thread sweeps
// whole pencils in registers.
//
// The pencil length is a run-time number, but each sweep runs code for exactly
// that length (a switch over 2 to LMAX, uniform over the launch; LMAX 8 for grids
// of short axes, whose 64 registers leave room for more one-wave blocks: 4^3
// 300x200 cells FP32 66 us against 81, FP64 87 against 156): a pencil of 20 cells in code
// for 32 with a window shifted by K, guards on every cell and unmerged
// differences took 3.5 times the instructions.  The first v_x sweep reads its
// pencils from global memory and the last writes them there (unit stride over
// the lanes), which saves two passes through shared memory and a barrier.
// 100 x 50 cells of 20x16x24 FP32: 578 us with one kernel for all lengths up
// to 32, 131 this way (2.3 TB/s).  Bound by its vector instructions (13 per cell and sweep
// besides the address of each access).

// Partial flux factor of a cell with value w between neighbours at distance dm
// below and dp above: phi = a X (the limited parabola of pfc_phi, the same
// operations: results as if it were called).
template <class T>
__device__ __forceinline__ T flux_factor(T w, T dm, T dp, T c1, T c2, T finf) {
    const T room = fmax(finf, w) - w;
    const T w2 = w + w, r2 = room + room;
    const T lp = med3(dp, -r2, w2), lm = med3(dm, -w2, r2);
    return fma(lm, c2, fma(lp, c1, w));
}

// Sub-cell sweep of a pencil in registers, in its direction of motion.
template <class T, int N>
__device__ __forceinline__ void sweep_exact(T (&g)[N], T a, T c1, T c2, T finf) {
#pragma clang fp contract(off)
    T dm = g[0];                 // g_m - g_{m-1}, zero ghost below
    T X = T(0), phi_prev = T(0);
#pragma unroll
    for (int m = 0; m < N - 1; ++m) {
        const T dp = g[m + 1] - g[m];
        X = flux_factor(g[m], dm, dp, c1, c2, finf);
        const T phi = X * a;
        g[m] = fmax((g[m] + phi_prev) - phi, T(0));
        phi_prev = phi;
        dm = dp;
    }
    g[N - 1] = fmax(fma(X, a, g[N - 1]), T(0));      // the wall face carries no flux
}

// A pencil in shared memory that moves by K >= 1 cells (element k at
// first + k step, downwind order), in place: cell p reads cells p - K - 2 ..
// p - K + 1, held in registers as a window; the wall cell keeps all that
// reaches it.  Code for each length up to 12, called: 60000 cells of 4^3 FP64
// moving by several cells 141 us, 199 with the loop below.
template <class T, int N>
__device__ __attribute__((noinline)) void pencil_far(LdsPtr<T> blk, int first, int step, int K, T a, T c1, T c2,
                                                      T finf) {
#pragma clang fp contract(off)
    T W[N + 2];                                       // W[j + 2]: cell j - K
    int q = first - (K + 2) * step;
#pragma unroll
    for (int j = -2; j < N; ++j) {
        const bool in = j - K >= 0;
        const T v = blk[in ? q : first];
        W[j + 2] = in ? v : T(0);
        q += step;
    }
    T top = T(0);
    for (int m = N - 1 - K > 0 ? N - 1 - K : 0; m < N; ++m) top += blk[first + m * step];
    auto factor = [&](int p) {                        // cell p - K
        const T w = W[p + 2];
        return flux_factor(w, w - W[p + 1], W[p + 3] - w, c1, c2, finf);
    };
    T X = factor(-1);
    T below = X * a;
#pragma unroll
    for (int p = 0; p < N - 1; ++p) {
        X = factor(p);
        const T phi = X * a;
        blk[first + p * step] = fmax((W[p + 2] + below) - phi, T(0));
        below = phi;
    }
    blk[first + (N - 1) * step] = fmax(fma(X, a, top), T(0));
}

// The same for longer pencils (n > 12) by a loop from the far end: output p reads
// cells up to p - K + 1, which outputs below p have not overwritten.  In a step
// the corner velocities of a block alone move by a cell, and a wave with one
// such pencil runs all of pencil_far beside the sub-cell code: steps of
// 100x50x20x16x24 FP32 855 us with it, 844 with the loop, 90x60x28x18x15 995 and
// 989.  Where most pencils move by cells (V alone, tau of hundreds of steps), the
// loop is slower: 20x16x24 262 and 315, FP64 10^3 230 and 413.
template <class T>
__device__ __attribute__((noinline)) void pencil_loop(LdsPtr<T> blk, int first, int step, int n, int K, T a,
                                                       T c1, T c2, T finf) {
#pragma clang fp contract(off)
    auto val = [&](int k) -> T { return k >= 0 ? blk[first + k * step] : T(0); };
    auto factor = [&](int k) {
        const T w = val(k);
        return flux_factor(w, w - val(k - 1), val(k + 1) - w, c1, c2, finf);
    };
    T top = T(0);
    for (int m = n - 1 - K > 0 ? n - 1 - K : 0; m < n; ++m) top += val(m);
    T X = factor(n - 2 - K);
    const T wall = fmax(fma(X, a, top), T(0));
    T phi = X * a;                                    // leaving window position p = n - 2
    for (int p = n - 2; p >= 0; --p) {
        const T w = val(p - K);
        X = factor(p - 1 - K);
        const T below = X * a;
        // the cells at and above p are read by no later output
        const T o = fmax((w + below) - phi, T(0));
        blk[first + p * step] = o;
        phi = below;
    }
    blk[first + (n - 1) * step] = wall;
}

// One pencil of N cells: kIn from global memory (else from shared), kOut to
// global memory (else back to shared).  Element m lives at first + m step in
// shared and goff + m gstep in global memory, in the direction of motion.
template <class T, int N, bool kIn, bool kOut>
__device__ __forceinline__ void pencil_exact(const T* __restrict__ src, T* __restrict__ dst, T* blk, unsigned goff,
                                             unsigned gstep, int first, int step, const Shift<T>& sh, T finf, T& mx) {
    T g[N];
    if constexpr (kIn) {
#pragma unroll
        for (int m = 0; m < N; ++m) g[m] = src[goff + (unsigned)m * gstep];
    } else {
#pragma unroll
        for (int m = 0; m < N; ++m) g[m] = blk[first + m * step];
    }
    if (sh.K == 0) {
        sweep_exact<T, N>(g, sh.a, sh.c1, sh.c2, finf);
        if constexpr (!kOut) {
#pragma unroll
            for (int m = 0; m < N; ++m) blk[first + m * step] = g[m];
        }
    } else {
        // beyond n + 2 cells every output but the wall cell is 0 either way
        const int K = sh.K > (long long)(N + 2) ? N + 2 : (int)sh.K;
        if constexpr (kIn) {
#pragma unroll
            for (int m = 0; m < N; ++m) blk[first + m * step] = g[m];
        }
        if constexpr (N <= 12)
            pencil_far<T, N>(lds_ptr(blk), first, step, K, sh.a, sh.c1, sh.c2, finf);
        else
            pencil_loop<T>(lds_ptr(blk), first, step, N, K, sh.a, sh.c1, sh.c2, finf);
        if constexpr (kOut) {
#pragma unroll
            for (int m = 0; m < N; ++m) g[m] = blk[first + m * step];
        }
    }
    if constexpr (kOut) {
#pragma unroll
        for (int m = 0; m < N; ++m) {
            dst[goff + (unsigned)m * gstep] = g[m];
            mx = fmax(mx, g[m]);
        }
    }
}

template <class T, bool kIn, bool kOut, int LMAX>
__device__ __forceinline__ void sweep_any(const T* __restrict__ src, T* __restrict__ dst, T* blk, int d, double sigma,
                                          const V3Params& P, const double (&EB)[6], T finf, T& mx) {
    const int pz = P.nvz | 1;
    const int n = d == 0 ? P.nvx : (d == 1 ? P.nvy : P.nvz);
    const int npen = d == 0 ? P.nvy * P.nvz : (d == 1 ? P.nvx * P.nvz : P.nvx * P.nvy);
    const int n2 = d == 2 ? P.nvy : P.nvz;            // second transverse axis
    const float inv_n2 = d == 2 ? P.inv_nvy : P.inv_nvz;
    for (int pen = threadIdx.x; pen < npen; pen += blockDim.x) {
        const int i1 = row_of(pen, inv_n2), i2 = pen - i1 * n2;
        int base, stride;
        double acc;
        if (d == 0) {           // pencil (iy, iz)
            base = i1 * pz + i2;
            stride = P.nvy * pz;
            const double vy = P.lo[1] + (i1 + 0.5) * P.dv[1], vz = P.lo[2] + (i2 + 0.5) * P.dv[2];
            acc = EB[0] + vy * EB[5] - vz * EB[4];
        } else if (d == 1) {    // pencil (ix, iz)
            base = i1 * P.nvy * pz + i2;
            stride = pz;
            const double vx = P.lo[0] + (i1 + 0.5) * P.dv[0], vz = P.lo[2] + (i2 + 0.5) * P.dv[2];
            acc = EB[1] + vz * EB[3] - vx * EB[5];
        } else {                // pencil (ix, iy)
            base = (i1 * P.nvy + i2) * pz;
            stride = 1;
            const double vx = P.lo[0] + (i1 + 0.5) * P.dv[0], vy = P.lo[1] + (i2 + 0.5) * P.dv[1];
            acc = EB[2] + vx * EB[4] - vy * EB[3];
        }
        const double s = P.qm * acc * sigma * P.inv_dv[d];
        const bool pos = s >= 0.0;
        const Shift<T> sh(fabs(s));
        const int first = pos ? base : base + (n - 1) * stride;
        const int step = pos ? stride : -stride;
        const unsigned plane = (unsigned)(P.nvy * P.nvz);
        const unsigned goff = pos ? (unsigned)pen : (unsigned)pen + (unsigned)(n - 1) * plane;
        const unsigned gstep = pos ? plane : 0u - plane;
#define VL_LEN(N)                                                                                     \
    case N:                                                                                           \
        if constexpr (N <= LMAX)                                                                      \
            pencil_exact<T, N, kIn, kOut>(src, dst, blk, goff, gstep, first, step, sh, finf, mx);     \
        break;
        VL_LENGTHS(n)
#undef VL_LEN
    }
}

template <class T, int LMAX, int NTH>
__global__ void __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(LMAX <= 8 ? (sizeof(T) == 4 ? 8 : 5) : (sizeof(T) == 4 ? 4 : 2))))
pfc_v3_kernel(const T* fin, T* fout, const double* __restrict__ E, const double* __restrict__ B,
              V3Params P, MaxRef finf_r, typename Bits<T>::U* __restrict__ max_out) {
    extern __shared__ unsigned char smem_raw[];
    T* blk = reinterpret_cast<T*>(smem_raw);
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const int nv = P.nvx * P.nvy * P.nvz;
    const T finf = max_of<T, true>(finf_r);
    double eb[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        eb[k] = E[cell * 3 + k];
        eb[3 + k] = B ? B[cell * 3 + k] : 0.0;
    }
    const T* src = fin + cell * nv;
    T* dst = fout + cell * nv;
    const double half = 0.5 * P.tau;
    T mx = T(0);
    sweep_any<T, true, false, LMAX>(src, dst, blk, 0, half, P, eb, finf, mx);
    __syncthreads();
    // one copy of the in-block code: vy, vz, vy
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        const int d = k == 1 ? 2 : 1;
        sweep_any<T, false, false, LMAX>(src, dst, blk, d, d == 2 ? P.tau : half, P, eb, finf, mx);
        __syncthreads();
    }
    sweep_any<T, false, true, LMAX>(src, dst, blk, 0, half, P, eb, finf, mx);
    if (max_out) block_max_part(mx, max_out);
}

// ---------------------------------------------------------------------------
// The same operator for cubic velocity blocks with compile-time edge N: every
// pencil has length N and a stride known at compile time, so a pencil is
// straight-line code with constant shared-memory offsets.
//
// The block is stored [v_x][v_y][v_z] with v_z padded to N | 1; a wave takes
// 64 / N values of the first transverse index and all of the second.
//
// Sub-cell shifts (K = 0, the common case): with D_m = g_m - g_{m-1} (zero
// ghosts), r2 = 2 f_inf - 2 g_m and
//   A_m = med3(D_{m+1}, -r2, 2 g_m),  B_m = med3(D_m, -2 g_m, r2),
// the partial flux leaving cell m downwind is a g_m + a c1 A_m + a c2 B_m for
// s > 0 and, by reflecting the pencil, a g_m - a c1 B_m - a c2 A_m for s < 0.
// The flux through face m+1/2 (positive towards m+1) is the first for cell m
// or minus the second for cell m+1; the wall faces carry none.
//
// Every sweep keeps 0 <= g <= f_inf, so 2 f_inf - 2 g_m >= 0 up to rounding
// and r2 is taken without its clamp at zero: where rounding puts g_m an ulp
// above f_inf the bound moves by that ulp.  A wave whose pencils all shift the
// same way walks them in the downwind order (a negative shift reads the
// pencil backwards, which with constant offsets costs nothing): one
// difference, seven operations for the partial flux and three for the update
// per element.  A wave with both signs keeps the storage order and selects
// per lane, one operation more.

// Sub-cell sweep of a pencil held in registers (updated in place) whose
// wave's lanes all shift one way: REV walks it from its far end (s < 0), so
// the downwind direction is always +m.
template <class T, int N, bool REV>
__device__ __forceinline__ void regs_one_way(T (&g)[N], T a, T c1, T c2, T F2) {
    auto u = [&](int m) -> T& { return g[REV ? N - 1 - m : m]; };
    T Dm = u(0);                 // D_m = g_m - g_{m-1}, zero ghost below
    T Dp = u(1) - u(0);
    T Fprev = T(0);              // flux through the lower wall
#pragma unroll
    for (int m = 0; m < N; ++m) {
        T F = T(0);              // flux through face m+1/2 (none through the upper wall)
        const T w = u(m);
        if (m + 1 < N) {
            F = sub_cell_flux(w, Dm, Dp, a, c1, c2, F2);
            Dm = Dp;
            Dp = (m + 2 < N ? u(m + 2) : T(0)) - u(m + 1);
        }
        u(m) = fmax(w + Fprev - F, T(0));
        Fprev = F;
    }
}

// The same for a wave holding both signs: storage order, the sign folded
// into the coefficients and a per-lane select of the face flux.
template <class T, int N>
__device__ __forceinline__ void regs_mixed(T (&g)[N], bool pos, T a, T ac1, T ac2, T F2) {
    const T cA = pos ? ac1 : -ac2;
    const T cB = pos ? ac2 : -ac1;
    // phi_m: partial flux of cell m in the lane's direction
    T Dm = g[0];
    T Dp = g[1] - g[0];
    T phi_m = sub_cell_flux(g[0], Dm, Dp, a, cA, cB, F2);
    T Fprev = T(0);
#pragma unroll
    for (int m = 0; m < N; ++m) {
        T Fnext = T(0), phi_n = T(0);
        if (m + 1 < N) {
            Dm = Dp;
            Dp = (m + 2 < N ? g[m + 2] : T(0)) - g[m + 1];
            phi_n = sub_cell_flux(g[m + 1], Dm, Dp, a, cA, cB, F2);
            Fnext = pos ? phi_m : -phi_n;
        }
        g[m] = fmax(g[m] + Fprev - Fnext, T(0));
        Fprev = Fnext;
        phi_m = phi_n;
    }
}

// Shifts of a cell or more (any lane of the wave): windows gathered in the
// sweep direction, the cells within K of the far wall summed into it.
template <class T, int N, class Ptr>
__device__ __attribute__((noinline)) void pencil_shifted(Ptr blk, int first, int step, int K, T a, T ac1, T ac2,
                                                          T F2) {
    T W[N + 2];
    int q = first - (K + 2) * step;
#pragma unroll
    for (int j = -2; j < N; ++j) {
        const bool in = j - K >= 0;
        const T v = blk[in ? q : first];
        W[j + 2] = in ? v : T(0);
        q += step;
    }
    T top = T(0);
    for (int m = (N - 1 - K > 0 ? N - 1 - K : 0); m < N; ++m) top += blk[first + m * step];
    T D = W[1] - W[0];
    T Dn = W[2] - W[1];
    T phi_prev = pfc_phi_d(W[1], D, Dn, a, ac1, ac2, F2);
    D = Dn;
    q = first;
#pragma unroll
    for (int p = 0; p < N - 1; ++p) {
        Dn = W[p + 3] - W[p + 2];
        const T phi_next = pfc_phi_d(W[p + 2], D, Dn, a, ac1, ac2, F2);
        blk[q] = fmax(W[p + 2] + phi_prev - phi_next, T(0));
        phi_prev = phi_next;
        D = Dn;
        q += step;
    }
    blk[q] = fmax(top + phi_prev, T(0));
}

// One PFC sweep of a pencil held in registers, its displacement split into
// its sign pos and the shift sh (cells).
// Shifts of a cell or more (any lane of the wave) go through the pencil's own
// cells blk[base + m stride] of the shared block, which no other thread
// touches meanwhile.
template <class T, int N>
__device__ __forceinline__ void sweep_pencil_regs(T (&g)[N], bool pos, const ShiftT<T>& sh, T F2, T* blk, int base,
                                                  int stride) {
    if (__all(sh.K == 0) && __all(pos)) {
        regs_one_way<T, N, false>(g, sh.a, sh.ac1, sh.ac2, F2);
    } else if (__all(sh.K == 0) && __all(!pos)) {
        regs_one_way<T, N, true>(g, sh.a, sh.ac1, sh.ac2, F2);
    } else if (__all(sh.K == 0)) {
        regs_mixed<T, N>(g, pos, sh.a, sh.ac1, sh.ac2, F2);
    } else {
#pragma unroll
        for (int m = 0; m < N; ++m) blk[base + m * stride] = g[m];
        const int K = sh.K > N + 2 ? N + 2 : sh.K;
        const int first = pos ? base : base + (N - 1) * stride;
        pencil_shifted<T, N>(lds_ptr(blk), first, pos ? stride : -stride, K, sh.a, sh.ac1, sh.ac2, F2);
#pragma unroll
        for (int m = 0; m < N; ++m) g[m] = blk[base + m * stride];
    }
}

// Displacement coefficients of sweep d: s = s0 + s1 i1 + s2 i2 over the
// pencil's two transverse indices (in FP64, then the storage type).
template <class T>
__device__ __forceinline__ void sweep_coeffs(int d, double sigma, const V3Params& P, const double* EB, T& s0, T& s1,
                                             T& s2) {
    const double C = P.qm * sigma * P.inv_dv[d];
    const double c0 = P.lo[0] + 0.5 * P.dv[0], c1 = P.lo[1] + 0.5 * P.dv[1], c2 = P.lo[2] + 0.5 * P.dv[2];
    double d0, d1, d2;
    if (d == 0) {           // pencil (iy, iz): a_x = (q/m)(Ex + vy Bz - vz By)
        d0 = C * (EB[0] + EB[5] * c1 - EB[4] * c2); d1 = C * EB[5] * P.dv[1]; d2 = -C * EB[4] * P.dv[2];
    } else if (d == 1) {    // pencil (ix, iz): a_y = (q/m)(Ey + vz Bx - vx Bz)
        d0 = C * (EB[1] + EB[3] * c2 - EB[5] * c0); d1 = -C * EB[5] * P.dv[0]; d2 = C * EB[3] * P.dv[2];
    } else {                // pencil (ix, iy): a_z = (q/m)(Ez + vx By - vy Bx)
        d0 = C * (EB[2] + EB[4] * c0 - EB[3] * c1); d1 = C * EB[4] * P.dv[0]; d2 = -C * EB[3] * P.dv[1];
    }
    s0 = (T)d0;
    s1 = (T)d1;
    s2 = (T)d2;
}

// One pencil of the cubic block along d (d = 0: (iy, iz); 1: (ix, iz); 2:
// (ix, iy)) with its shift split as pos / sh.
template <class T, int N>
__device__ __forceinline__ void sweep_cube_pencil(T* blk, int d, int pen, bool pos, const ShiftT<T>& sh, T F2) {
    constexpr int PZ = N | 1;
    const int stride = d == 0 ? N * PZ : (d == 1 ? PZ : 1);
    const int i1 = pen / N, i2 = pen % N;
    const int base = d == 0 ? i1 * PZ + i2 : (d == 1 ? i1 * N * PZ + i2 : (i1 * N + i2) * PZ);
    if (__all(sh.K == 0)) {
        T* pb = blk + base;
        T g[N];
#pragma unroll
        for (int m = 0; m < N; ++m) g[m] = pb[m * stride];
        if (__all(pos))
            regs_one_way<T, N, false>(g, sh.a, sh.ac1, sh.ac2, F2);
        else if (__all(!pos))
            regs_one_way<T, N, true>(g, sh.a, sh.ac1, sh.ac2, F2);
        else
            regs_mixed<T, N>(g, pos, sh.a, sh.ac1, sh.ac2, F2);
#pragma unroll
        for (int m = 0; m < N; ++m) pb[m * stride] = g[m];
    } else {
        const int K = sh.K > N + 2 ? N + 2 : sh.K;
        const int first = pos ? base : base + (N - 1) * stride;
        pencil_shifted<T, N>(lds_ptr(blk), first, pos ? stride : -stride, K, sh.a, sh.ac1, sh.ac2, F2);
    }
}

// Shift of pencil pen of sweep d from the sweep's coefficients.
template <class T, int N>
__device__ __forceinline__ T cube_pencil_shift(int pen, T s0, T s1, T s2) {
    return fma(s1, (T)(pen / N), fma(s2, (T)(pen % N), s0));
}

template <class T, int N>
__device__ __forceinline__ void sweep_cube(T* blk, int d, double sigma, const V3Params& P, const double* EB, T F2) {
    T s0, s1, s2;
    sweep_coeffs<T>(d, sigma, P, EB, s0, s1, s2);
    for (int pen = threadIdx.x; pen < N * N; pen += blockDim.x) {
        const T s = cube_pencil_shift<T, N>(pen, s0, s1, s2);
        sweep_cube_pencil<T, N>(blk, d, pen, s >= T(0), ShiftT<T>(fabs(s)), F2);
    }
}

template <class T, int N, int NTH, bool kFold>
__global__ void __launch_bounds__(NTH)
pfc_v3_cube_kernel(const T* fin, T* fout, const double* __restrict__ E, const double* __restrict__ B, V3Params P,
                   MaxRef finf_r, typename Bits<T>::U* __restrict__ max_out) {
    constexpr int PZ = N | 1;
    constexpr int NV = N * N * N;
    constexpr int PER = NV / NTH;            // values per thread (NTH divides N^3)
    static_assert(PER * NTH == NV, "thread count must divide the block");
    // one v_x pencil per thread, or two: the two v_x sweeps run in registers
    constexpr bool kRegX = N * N <= NTH;
    constexpr bool kRegX2 = !kRegX && N * N <= 2 * NTH;
    __shared__ T blk[N * N * PZ];
    __shared__ double EB[6];
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const T F2 = T(2) * max_of<T, kFold>(finf_r);
    if (threadIdx.x < 3) {
        EB[threadIdx.x] = E[cell * 3 + threadIdx.x];
        EB[3 + threadIdx.x] = B ? B[cell * 3 + threadIdx.x] : 0.0;
    }
    const double half = 0.5 * P.tau;
    const T* src = fin + cell * NV;
    T* dst = fout + cell * NV;
    T mx = T(0);
    if constexpr (kRegX) {
        // Thread t owns the v_x pencil at (iy, iz) = (t / N, t % N): it loads it
        // (unit stride across the wave), sweeps it, and stores it into the block
        // for the v_y, v_z, v_y sweeps; then reads it back for the last v_x
        // sweep and writes it out.  The fields come straight from global
        // memory for the first sweep, which runs before any barrier.
        const int t = threadIdx.x;
        const bool own = t < N * N;
        const int xb = (t / N) * PZ + t % N;
        constexpr int XS = N * PZ;
        double eb[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            eb[k] = E[cell * 3 + k];
            eb[3 + k] = B ? B[cell * 3 + k] : 0.0;
        }
        T xs0, xs1, xs2;
        sweep_coeffs<T>(0, half, P, eb, xs0, xs1, xs2);
        const T sx = fma(xs1, (T)(t / N), fma(xs2, (T)(t % N), xs0));
        const bool posx = sx >= T(0);
        const ShiftT<T> shx(fabs(sx));         // both v_x sweeps
        T g[N];
        if (own) {
#pragma unroll
            for (int k = 0; k < N; ++k) g[k] = __builtin_nontemporal_load(src + t + k * N * N);
            sweep_pencil_regs<T, N>(g, posx, shx, F2, blk, xb, XS);
#pragma unroll
            for (int k = 0; k < N; ++k) blk[xb + k * XS] = g[k];
        }
        __syncthreads();
        // one v_y and one v_z pencil per thread: their shifts are set up once,
        // the v_y one serving both v_y sweeps
        {
            T c0, c1, c2;
            sweep_coeffs<T>(1, half, P, EB, c0, c1, c2);
            const T sy = cube_pencil_shift<T, N>(t, c0, c1, c2);
            sweep_coeffs<T>(2, P.tau, P, EB, c0, c1, c2);
            const T sz = cube_pencil_shift<T, N>(t, c0, c1, c2);
            const ShiftT<T> shy(fabs(sy)), shz(fabs(sz));
            if (own) sweep_cube_pencil<T, N>(blk, 1, t, sy >= T(0), shy, F2);
            __syncthreads();
            if (own) sweep_cube_pencil<T, N>(blk, 2, t, sz >= T(0), shz, F2);
            __syncthreads();
            if (own) sweep_cube_pencil<T, N>(blk, 1, t, sy >= T(0), shy, F2);
            __syncthreads();
        }
        if (own) {
#pragma unroll
            for (int k = 0; k < N; ++k) g[k] = blk[xb + k * XS];
            sweep_pencil_regs<T, N>(g, posx, shx, F2, blk, xb, XS);
#pragma unroll
            for (int k = 0; k < N; ++k) {
                __builtin_nontemporal_store(g[k], dst + t + k * N * N);
                mx = fmax(mx, g[k]);
            }
        }
    } else if constexpr (kRegX2) {
        // Thread t owns the v_x pencils t and t + NTH (those below N^2): each is
        // loaded from global memory, swept in registers and stored into the
        // block; after the v_y, v_z, v_y sweeps in the block each is read back,
        // swept again and written out.  One pencil is in registers at a time.
        // A 34^3 v_x plane is not a whole number of lines (4624 B in FP32):
        // ordinary loads and stores let the caches merge the lines two wave
        // accesses share (4.01 -> 3.83 ms per 256x128x34^3 launch).
        const int t = threadIdx.x;
        constexpr int XS = N * PZ;
        double eb[6];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            eb[k] = E[cell * 3 + k];
            eb[3 + k] = B ? B[cell * 3 + k] : 0.0;
        }
        T xs0, xs1, xs2;
        sweep_coeffs<T>(0, half, P, eb, xs0, xs1, xs2);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = t + j * NTH;
            if (p < N * N) {
                const int xb = (p / N) * PZ + p % N;
                const T sx = cube_pencil_shift<T, N>(p, xs0, xs1, xs2);
                T g[N];
#pragma unroll
                for (int k = 0; k < N; ++k) g[k] = ld_f<kRowsWholeLines<T, N>>(src + p + k * N * N);
                sweep_pencil_regs<T, N>(g, sx >= T(0), ShiftT<T>(fabs(sx)), F2, blk, xb, XS);
#pragma unroll
                for (int k = 0; k < N; ++k) blk[xb + k * XS] = g[k];
            }
        }
        __syncthreads();
        sweep_cube<T, N>(blk, 1, half, P, EB, F2);
        __syncthreads();
        sweep_cube<T, N>(blk, 2, P.tau, P, EB, F2);
        __syncthreads();
        sweep_cube<T, N>(blk, 1, half, P, EB, F2);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = t + j * NTH;
            if (p < N * N) {
                const int xb = (p / N) * PZ + p % N;
                const T sx = cube_pencil_shift<T, N>(p, xs0, xs1, xs2);
                T g[N];
#pragma unroll
                for (int k = 0; k < N; ++k) g[k] = blk[xb + k * XS];
                sweep_pencil_regs<T, N>(g, sx >= T(0), ShiftT<T>(fabs(sx)), F2, blk, xb, XS);
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    st_f<kRowsWholeLines<T, N>>(g[k], dst + p + k * N * N);
                    mx = fmax(mx, g[k]);
                }
            }
        }
    } else {
        // large blocks stream through registers in chunks of four values per
        // thread
        constexpr int CH = PER > 16 ? 4 : PER;
        static_assert(PER % CH == 0, "chunks must tile the block");
#pragma unroll 1
        for (int c0 = 0; c0 < PER; c0 += CH) {
            T v[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) v[j] = __builtin_nontemporal_load(src + threadIdx.x + (c0 + j) * NTH);
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int e = threadIdx.x + (c0 + j) * NTH;
                blk[e + (e / N) * (PZ - N)] = v[j];
            }
        }
        __syncthreads();
        // each sweep reads the fields from shared memory after its barrier, which
        // keeps the five sweeps' shift set-ups from being hoisted (and held live)
        sweep_cube<T, N>(blk, 0, half, P, EB, F2);
        __syncthreads();
        sweep_cube<T, N>(blk, 1, half, P, EB, F2);
        __syncthreads();
        sweep_cube<T, N>(blk, 2, P.tau, P, EB, F2);
        __syncthreads();
        sweep_cube<T, N>(blk, 1, half, P, EB, F2);
        __syncthreads();
        sweep_cube<T, N>(blk, 0, half, P, EB, F2);
        __syncthreads();
#pragma unroll 1
        for (int c0 = 0; c0 < PER; c0 += CH) {
            T v[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int e = threadIdx.x + (c0 + j) * NTH;
                v[j] = blk[e + (e / N) * (PZ - N)];
            }
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                __builtin_nontemporal_store(v[j], dst + threadIdx.x + (c0 + j) * NTH);
                mx = fmax(mx, v[j]);
            }
        }
    }
    if (max_out) block_max_part(mx, max_out);
}

// ---------------------------------------------------------------------------
// The same operator when the block is larger than a CU's shared memory (the
// FP64 34^3 block, 314 KB, against 160 KB).  The v_y, v_z, v_y sweeps stay
// inside the planes of fixed v_x, so they run on PL planes at a time in shared
// memory (N / PL = 2 rounds); the rest of the block waits in registers.
// Thread t owns the v_x pencils p = t + NTH j (p < N^2):
//  1. each pencil is loaded, swept along v_x in registers, and split: its
//     values in the first PL planes go to shared memory, the others wait in
//     registers (a[j]; those of the partial last pencil set, which only some
//     threads own, in the pencil's own positions of the output block);
//  2. round 0 sweeps the first PL planes; each thread then swaps its own
//     plane values with a[j] (no other thread touches them), and round 1
//     sweeps the last PL planes;
//  3. each pencil is reassembled from a[j] and shared memory, swept along v_x
//     again and stored.
// Eight waves per block leave 256 registers per lane.  A v_x pencil that
// shifts by a cell or more is swept in the cell's output block, in its own
// positions, which nothing else reads or writes meanwhile (in place as well:
// the pencil's input has been read by then).
template <class T, int N, int NTH, int PL, bool kFold>
__global__ void __launch_bounds__(NTH)
pfc_v3_planes_kernel(const T* fin, T* fout, const double* __restrict__ E, const double* __restrict__ B,
                     V3Params P, MaxRef finf_r, typename Bits<T>::U* __restrict__ max_out) {
    constexpr int PZ = N | 1;
    constexpr int NN = N * N;
    constexpr int NP = (NN + NTH - 1) / NTH;     // v_x pencils per thread (the last one partial)
    constexpr unsigned XB = NN * sizeof(T);      // bytes between v_x planes
    static_assert(2 * PL == N, "two rounds of PL planes");
    static_assert(NN <= NP * NTH, "pencils cover the block");
    __shared__ T blk[PL * N * PZ];
    const int t = threadIdx.x;
    const long long cell = xcd_work_index(blockIdx.x, gridDim.x);
    const T F2 = T(2) * max_of<T, kFold>(finf_r);
    T* dst = fout + cell * (N * NN);
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(fin + cell * (N * NN)), 0, N * XB, kBufWord3);
    const auto rd = __builtin_amdgcn_make_buffer_rsrc(dst, 0, N * XB, kBufWord3);
    double eb[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        eb[k] = E[cell * 3 + k];
        eb[3 + k] = B ? B[cell * 3 + k] : 0.0;
    }
    const double half = 0.5 * P.tau;
    T xs0, xs1, xs2, y0, y1, y2, z0, z1, z2;
    sweep_coeffs<T>(0, half, P, eb, xs0, xs1, xs2);
    sweep_coeffs<T>(1, half, P, eb, y0, y1, y2);
    sweep_coeffs<T>(2, P.tau, P, eb, z0, z1, z2);
    // v_x sweep of pencil p held in g; shifts of a cell or more go through the
    // pencil's own positions of the output block
    auto sweep_x = [&](T (&g)[N], int p) {
        const T sx = cube_pencil_shift<T, N>(p, xs0, xs1, xs2);
        const bool pos = sx >= T(0);
        const ShiftT<T> sh(fabs(sx));
        if (__all(sh.K == 0) && __all(pos)) {
            regs_one_way<T, N, false>(g, sh.a, sh.ac1, sh.ac2, F2);
        } else if (__all(sh.K == 0) && __all(!pos)) {
            regs_one_way<T, N, true>(g, sh.a, sh.ac1, sh.ac2, F2);
        } else if (__all(sh.K == 0)) {
            regs_mixed<T, N>(g, pos, sh.a, sh.ac1, sh.ac2, F2);
        } else {
            const unsigned po = (unsigned)p * sizeof(T);
#pragma unroll
            for (int m = 0; m < N; ++m) buf_st(g[m], rd, po, m * XB);
            const int K = sh.K > N + 2 ? N + 2 : sh.K;
            const int first = pos ? p : p + (N - 1) * NN;
            pencil_shifted<T, N>(dst, first, pos ? NN : -NN, K, sh.a, sh.ac1, sh.ac2, F2);
#pragma unroll
            for (int m = 0; m < N; ++m) g[m] = buf_ld(rd, po, m * XB, T());
        }
    };
    // the last plane halves of the full pencils wait in registers, those of
    // the partial last pencil (NN - (NP - 1) NTH of them) in its own
    // positions of the output block
    T a[NP - 1][PL];
    // 1. v_x half sweep; the first PL planes to shared memory
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int p = t + NTH * j;
        if (p < NN) {
            const int o = (p / N) * PZ + p % N;
            const unsigned po = (unsigned)p * sizeof(T);
            T g[N];
#pragma unroll
            for (int k = 0; k < N; ++k) g[k] = buf_ld(rs, po, k * XB, T());
            sweep_x(g, p);
#pragma unroll
            for (int k = 0; k < PL; ++k) {
                blk[k * N * PZ + o] = g[k];
                if (j < NP - 1)
                    a[j < NP - 1 ? j : 0][k] = g[PL + k];
                else
                    buf_st(g[PL + k], rd, po, (PL + k) * XB);
            }
        }
    }
    // 2. in-plane sweeps, round r on planes r PL .. r PL + PL - 1
    auto in_plane = [&](int r) {
        for (int pen = t; pen < PL * N; pen += NTH) {
            const int pg = pen + r * PL * N;        // (v_x plane, second index) over the whole block
            const T sy = cube_pencil_shift<T, N>(pg, y0, y1, y2);
            sweep_cube_pencil<T, N>(blk, 1, pen, sy >= T(0), ShiftT<T>(fabs(sy)), F2);
        }
        __syncthreads();
        for (int pen = t; pen < PL * N; pen += NTH) {
            const int pg = pen + r * PL * N;
            const T sz = cube_pencil_shift<T, N>(pg, z0, z1, z2);
            sweep_cube_pencil<T, N>(blk, 2, pen, sz >= T(0), ShiftT<T>(fabs(sz)), F2);
        }
        __syncthreads();
        for (int pen = t; pen < PL * N; pen += NTH) {
            const int pg = pen + r * PL * N;
            const T sy = cube_pencil_shift<T, N>(pg, y0, y1, y2);
            sweep_cube_pencil<T, N>(blk, 1, pen, sy >= T(0), ShiftT<T>(fabs(sy)), F2);
        }
        __syncthreads();
    };
    __syncthreads();
    in_plane(0);
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int p = t + NTH * j;
        if (p < NN) {
            const int o = (p / N) * PZ + p % N;
            const unsigned po = (unsigned)p * sizeof(T);
#pragma unroll
            for (int k = 0; k < PL; ++k) {
                const T v = blk[k * N * PZ + o];
                if (j < NP - 1) {
                    blk[k * N * PZ + o] = a[j < NP - 1 ? j : 0][k];
                    a[j < NP - 1 ? j : 0][k] = v;
                } else {
                    blk[k * N * PZ + o] = buf_ld(rd, po, (PL + k) * XB, T());
                    buf_st(v, rd, po, k * XB);
                }
            }
        }
    }
    __syncthreads();
    in_plane(1);
    // 3. second v_x half sweep and the store
    T mx = T(0);
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int p = t + NTH * j;
        if (p < NN) {
            const int o = (p / N) * PZ + p % N;
            const unsigned po = (unsigned)p * sizeof(T);
            T g[N];
#pragma unroll
            for (int k = 0; k < PL; ++k) {
                g[k] = j < NP - 1 ? a[j < NP - 1 ? j : 0][k] : buf_ld(rd, po, k * XB, T());
                g[PL + k] = blk[k * N * PZ + o];
            }
            sweep_x(g, p);
#pragma unroll
            for (int k = 0; k < N; ++k) {
                buf_st(g[k], rd, po, k * XB);
                mx = fmax(mx, g[k]);
            }
        }
    }
    if (max_out) block_max_part(mx, max_out);
}

// ---------------------------------------------------------------------------
// Maximum of an array: 16-byte loads (where f is 16-byte aligned), four in
// flight per thread.  Read past the caches where f is larger than the last-level
// cache (226 MB: 58 us with one 4-byte load in flight, 48 with 16-byte loads
// through the caches, 38 past them, 6.0 TB/s), else through it: the operator
// that needs the maximum reads f next and gains more than this kernel loses.
// X and its maximum, FP64 8^3 256x128 (134 MB) 103 us past and 94 through the
// caches, FP32 10^3 200x100 (80 MB) 72 and 67, 12^3 at 224 MB 158 and 151;
// beyond, V or X of 268 to 450 MB is 1 to 5 % slower through them, and
// backsubstitution at 226 MB 194 against 190.
constexpr long long kLastLevelBytes = 208ll << 20;
template <class T, bool kPast>
__global__ void __launch_bounds__(256)
array_max_kernel(const T* __restrict__ f, long long n, typename Bits<T>::U* __restrict__ out) {
    constexpr int V = 16 / (int)sizeof(T);
    typedef T Vec __attribute__((ext_vector_type(V)));
    T mx = T(0);
    const long long stride = (long long)gridDim.x * 256, at = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long nvec = ((uintptr_t)f & 15u) ? 0 : n / V;
    const Vec* fv = reinterpret_cast<const Vec*>(f);
    long long i = at;
    for (; i + 3 * stride < nvec; i += 4 * stride) {
        Vec v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if constexpr (kPast) v[u] = __builtin_nontemporal_load(fv + i + u * stride);
            else v[u] = fv[i + u * stride];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < V; ++k) mx = fmax(mx, v[u][k]);
    }
    for (; i < nvec; i += stride) {
        const Vec v = fv[i];
#pragma unroll
        for (int k = 0; k < V; ++k) mx = fmax(mx, v[k]);
    }
    for (i = nvec * V + at; i < n; i += stride) mx = fmax(mx, f[i]);
    block_max_part(mx, out);
}

// Maximum of the per-block partial maxima part[0..n) into *slot (bits of
// non-negative values order like the values).  Up to kFoldOne partials: one
// 1024-thread block, 16-byte loads, eight in flight per thread (32768 FP32
// partials: 13.2 us in the two launches below, 4.8 us in one).  More: up to
// kFinStage blocks each fold a contiguous range of the partials (eight loads
// in flight per thread) into stage[b], placed right after the partials
// (fin_stage), and one wave folds the stage into the slot: 2 MB of partials
// are more than one CU reads quickly (524288: 10.7 + 4.7 us).  Fixed order.
template <class U>
__global__ void __launch_bounds__(1024)
max_fold_kernel(const U* __restrict__ part, int n, U* __restrict__ slot) {
    fold_max_block<U>(part, n, slot);
}

template <class U>
__global__ void __launch_bounds__(256)
max_stage_kernel(const U* __restrict__ part, long long n, long long chunk, U* __restrict__ out) {
    __shared__ U red[256 / kWave];
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = lo + chunk < n ? lo + chunk : n;
    U m = 0;
    for (long long b = lo; b < hi; b += 8 * 256) {
        U v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long long i = b + u * 256 + threadIdx.x;
            v[u] = i < hi ? part[i] : U(0);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) m = v[u] > m ? v[u] : m;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const U y = __shfl_xor(m, o, kWave);
        m = y > m ? y : m;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / kWave; ++w) m = red[w] > m ? red[w] : m;
        out[blockIdx.x] = m;
    }
}

template <class U>
__global__ void __launch_bounds__(kWave) max_final_kernel(const U* __restrict__ stage, int g, U* __restrict__ slot) {
    U m = (int)threadIdx.x < g ? stage[threadIdx.x] : U(0);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const U y = __shfl_xor(m, o, kWave);
        m = y > m ? y : m;
    }
    if (threadIdx.x == 0) *slot = m;
}

template <class T>
hipError_t launch_max_finalize(const void* part, long long n, void* slot, hipStream_t st) {
    using U = typename Bits<T>::U;
    if (n <= kFoldOne) {
        hipLaunchKernelGGL((max_fold_kernel<U>), dim3(1), dim3(1024), 0, st, (const U*)part, (int)n, (U*)slot);
        return hipGetLastError();
    }
    const FinSplit fs = fin_split(n);
    U* stage = (U*)((char*)part + fin_stage(n, sizeof(U)));
    hipLaunchKernelGGL((max_stage_kernel<U>), dim3(fs.blocks), dim3(256), 0, st, (const U*)part, n, fs.chunk, stage);
    hipLaunchKernelGGL((max_final_kernel<U>), dim3(1), dim3(kWave), 0, st, (const U*)stage, fs.blocks, (U*)slot);
    return hipGetLastError();
}

// ------------------------------------------------------------ launchers ----
// A launcher given a sink has its kernel store per-block maxima in it (in the
// slot itself where they fit, else in the sink's partials, which it then
// reduces into the slot).
constexpr int kChunkX = 16;

long long pfc_x_blocks(int rows, int nx, long long Nv) { return ((Nv + 255) / 256) * ((nx + kChunkX - 1) / kChunkX) * rows; }

template <class T>
static hipError_t finish_max(const MaxSink& sink, long long blocks, hipStream_t st) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !sink.slot || sink.direct(blocks)) return e;
    return launch_max_finalize<T>(sink.part, blocks, sink.slot, st);
}

template <class T>
hipError_t launch_pfc_x(const T* fin, T* fout, int rows, int nx, long long Nv, int inner, double vx_lo,
                        double dvx, double tau_dx, MaxRef finf, const MaxSink& sink, hipStream_t st) {
    const long long blocks = pfc_x_blocks(rows, nx, Nv);
    hipLaunchKernelGGL((finf.n > 1 ? pfc_x_kernel<T, kChunkX, true> : pfc_x_kernel<T, kChunkX, false>), dim3((unsigned)blocks), dim3(256), 0, st, fin, fout, nx, (int)Nv,
                       1.0f / (float)inner, vx_lo, dvx, tau_dx, finf,
                       sink.target<T>(blocks));
    return finish_max<T>(sink, blocks, st);
}

// x cells per thread: 8 in both storage types (FP64: 256 registers, one wave
// per SIMD, no spill; against 4 columns 3292 -> 3061 us per 1024x512x12^3
// launch and 456 -> 395 us per 256x128x16^3 launch; 12 columns: 3134 us),
// and 16 for FP32 velocity blocks of 64 KB or more (below)
template <class T> constexpr int xy_cols() { return 8; }
template <class T> constexpr int xy_cols_big() { return sizeof(T) == 4 ? 16 : 8; }

// Rows per segment of the fused X operator.  Waves in flight per CU the
// model assumes: 12 in FP32 (register-limited to 3 per SIMD), 8 in FP64 (the
// value the FP64 strip widths were measured with).  A wave walks
// S + 2 Kmax + 4 rows for S outputs.  Beyond the one-round case in
// xy_segment, the model cost rounds(S) * (S + 4 + 2 Kmax), with rounds the
// number of times the waves of the launch refill the GPU, picks the segment
// count (at most 64, segments of at least 8 rows; of at least 4 where the waves
// then still have a SIMD each).
static int xy_cus() {
    static int cus = 0;
    if (cus <= 0) {
        int d = 0;
        if (hipGetDevice(&d) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, d) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}
constexpr int kXyMaxSeg = 64;
constexpr size_t kXyCached = (size_t)512 << 20;      // bytes of f
static int xy_segment(int ny, long long waves_per_seg, int kb, int waves_per_cu) {
    const long long resident = (long long)waves_per_cu * xy_cus();
    // segments of 128 rows that fill at least half the GPU in one round: one
    // round of long walks (GEM 256x128x16^3: 200 us per launch against 212
    // for the two rounds of 43-row segments the cost model picks)
    const int s128 = ny < 128 ? ny : 128;
    const long long w128 = waves_per_seg * ((ny + s128 - 1) / s128);
    if (w128 <= resident && 2 * w128 >= resident) return s128;
    int bestS = ny;
    double best = 0.0;
    for (int n = 1; n <= kXyMaxSeg && n <= ny; ++n) {
        const int S = (ny + n - 1) / n;
        if ((ny + S - 1) / S != n) continue;      // the same split as a smaller n
        const long long w = waves_per_seg * n;
        if (n > 1 && S < (w <= 4 * xy_cus() ? 4 : 8)) break;
        const double cost = (double)((w + resident - 1) / resident) * (double)(S + 4 + 2 * kb);
        if (n == 1 || cost < best * 0.999) {
            best = cost;
            bestS = S;
        }
    }
    return bestS;
}

static long long xy_waves_per_seg(int nx, long long Nv, int cols) {
    return ((Nv + kWave - 1) / kWave) * ((nx + cols - 1) / cols);
}

// Bound of the whole-cell y shift (one more than the FP64 estimate: the
// kernel splits the shift in the storage type).
static int xy_ky_bound(int ny, int nvy, double vy_lo, double dvy, double tau_dy, int per) {
    const double vymax = fmax(fabs(vy_lo), fabs(vy_lo + nvy * dvy));
    const double kd = floor(vymax * tau_dy) + 1.0;
    const int L = per ? ny : 2 * ny;
    return kd >= (double)L ? L - 1 : (int)kd;
}

template <class T>
static int xy_waves_per_cu(int cols) {
    return sizeof(T) == 4 ? (cols <= 4 ? 16 : 12) : 8;
}

// Mean over largest number of waves a SIMD gets from the launch with `cols`
// columns.
template <class T>
static double xy_even(int nx, int ny, long long Nv, int kb, int cols) {
    const long long w1 = xy_waves_per_seg(nx, Nv, cols), simds = 4LL * xy_cus();
    const int S = xy_segment(ny, w1, kb, xy_waves_per_cu<T>(cols));
    const long long w = w1 * ((ny + S - 1) / S);
    return (double)w / (double)((w + simds - 1) / simds * simds);
}

// Upper bound of the launch's blocks over every strip width and segment length
// it can pick, for any tau (sizes the per-block partial maxima).
long long pfc_xy_blocks(int nx, int ny, int nvx, int nvy, int nvz) {
    const long long Nv = (long long)nvx * nvy * nvz;
    // more than one segment: S = ceil(ny / n) >= 4 in xy_segment, or 128 rows each
    const int most = ny > 4 ? (ny - 1) / 3 : 1;
    const long long nseg = most < kXyMaxSeg ? most : ((ny + 127) / 128 > kXyMaxSeg ? (ny + 127) / 128 : kXyMaxSeg);
    const long long w = xy_waves_per_seg(nx, Nv, 4) * nseg;    // 4 columns: a bound for every strip width
    return (w + 3) / 4;
}

template <class T, int C>
static hipError_t launch_pfc_xy_cols(const T* fin, T* fout, int nx, int ny, int nvx, int nvy, int nvz, double vx_lo,
                                     double dvx, double tau_dx, double vy_lo, double dvy, double tau_dy, int per,
                                     MaxRef finf, const MaxSink& sink, hipStream_t st) {
    XYArgs A;
    A.nx = nx;
    A.ny = ny;
    A.Nv = nvx * nvy * nvz;
    A.nvy = nvy;
    A.nvz = nvz;
    A.per = per;
    A.inv_nvz = 1.0f / (float)nvz;
    A.inv_nvyz = 1.0f / (float)(nvy * nvz);
    A.vx_lo = vx_lo;
    A.dvx = dvx;
    A.tau_dx = tau_dx;
    A.vy_lo = vy_lo;
    A.dvy = dvy;
    A.tau_dy = tau_dy;
    A.nchunks = (A.Nv + kWave - 1) / kWave;
    A.nst = (nx + C - 1) / C;
    const int kb = xy_ky_bound(ny, nvy, vy_lo, dvy, tau_dy, per);
    A.S = xy_segment(ny, xy_waves_per_seg(nx, A.Nv, C), kb, xy_waves_per_cu<T>(C));
    A.nseg = (ny + A.S - 1) / A.S;
    const long long waves = xy_waves_per_seg(nx, A.Nv, C) * A.nseg;
    const long long blocks = (waves + 3) / 4;
    // the stores of one step span rows i-2-Kmax .. i-1+Kmax of one pass
    const size_t rowbytes = (size_t)nx * A.Nv * sizeof(T);
    const bool wide = (double)(2 * kb + 3) * (double)rowbytes >= 4294967296.0;
    auto* mo = sink.target<T>(blocks);
    A.pad = mo && sink.direct(blocks) ? sink.fixed : 0;
    // Workgroups resident per CU, set through a reservation of shared memory
    // the kernel does not use: with fewer waves in flight the walks of large
    // velocity blocks thrash the caches and the address translation less.
    // Measured per launch (FP32): 34^3 blocks (157 KB per cell) one workgroup
    // per CU, 12.9 -> 11.0 ms on 512x256; blocks of at most 8 KB (12^3) two,
    // 1.70 -> 1.57 ms on 1024x512 and 0.42 -> 0.41 on 512x256 (906 MB), but only
    // where f is far beyond the caches: 8^3 on 512x256 (268 MB) 112 us without,
    // 124 with, and 256x128 (67 MB) 35 and 41; 16^3 unchanged with the register
    // limit's three (two: +1 %, one: +33 %).
    const size_t cellb = (size_t)A.Nv * sizeof(T);
    const size_t shm = cellb >= 65536 ? 102400 : (cellb <= 8192 && rowbytes * ny >= kXyCached ? 61440 : 0);
    if (wide)
        hipLaunchKernelGGL((finf.n > 1 ? pfc_xy_kernel<T, C, true, true> : pfc_xy_kernel<T, C, true, false>), dim3((unsigned)blocks), dim3(256), shm, st, fin, fout, A,
                           finf, mo);
    else
        hipLaunchKernelGGL((finf.n > 1 ? pfc_xy_kernel<T, C, false, true> : pfc_xy_kernel<T, C, false, false>), dim3((unsigned)blocks), dim3(256), shm, st, fin, fout, A,
                           finf, mo);
    return finish_max<T>(sink, blocks, st);
}

// Columns per lane: xy_cols for most blocks; for FP32 velocity blocks of 64 KB
// or more (34^3) twice that, where the wider strip's fewer halo loads per
// output pay for the registers (one wave per SIMD; the launcher keeps one
// workgroup per CU there anyway): 11.0 -> 10.2 ms per 512x256x34^3 FP32
// launch (FP64 34^3: 8 against 4 columns, 5.28 -> 4.68 ms per 256x128x34^3
// launch).  At 12^3 and 16^3 the wider FP32 strip is 3-18 % slower, and 4,
// 6, 10 or 12 columns are slower than 8 at 12^3 on large grids.  Small grids
// take 4: a wave's walk is a chain of rows whose length in time grows with the
// strip, and 8 columns leave SIMDs without a wave.  The line is a launch of
// kXyNarrow waves per CU at 4 columns and 8 rows.  Below it, per launch in a
// step: FP32 32x16x8^3 14.4 -> 8.5 us (with the shorter segments); per step: FP32
// 20x11x16^3 168 -> 139 us, 80x50x8^3 178 -> 168, FP64 32x16x12^3 192 -> 164; per
// call with the maximum of f: FP64 45x22x16^3 40 -> 31, 64x32x16^3 53 -> 47.
// Beyond it 8 columns win at 16^3 (FP64 128x64 154 against 162, FP32 256x128 315
// against 330), except where they deal the SIMDs uneven numbers of waves, which
// all walk a segment of the same length: 4 columns then if they are more even by
// a fifth.  Calls as above: FP32 100x50x20x16x24 (1560 waves of 8 columns on 1024
// SIMDs, 3000 of 4) 95 -> 89, FP64 100x50x20x16x18 187 -> 154; per step: FP64
// 100x50x20x16x18 1640 -> 1521, 180x90x16^3 2165 -> 2040, FP32 150x80x20x16x24
// 1925 -> 1871, 100x50x20x16x24 844 -> 842.  More even by less than a tenth: FP32
// 180x90x16^3 163 -> 167, FP64 150x80x20x16x18 354 -> 373 (calls).  Only below
// kXyCached bytes of f: beyond, what the caches hold decides.
constexpr int kXyNarrow = 16;
template <class T>
hipError_t launch_pfc_xy(const T* fin, T* fout, int nx, int ny, int nvx, int nvy, int nvz, double vx_lo, double dvx,
                         double tau_dx, double vy_lo, double dvy, double tau_dy, int per, MaxRef finf,
                         const MaxSink& sink, hipStream_t st) {
    const long long Nv = (long long)nvx * nvy * nvz;
    const size_t cellb = (size_t)Nv * sizeof(T);
    const int kb = xy_ky_bound(ny, nvy, vy_lo, dvy, tau_dy, per);
    if (cellb < 65536 &&
        (xy_waves_per_seg(nx, Nv, 4) * ((ny + 7) / 8) <= (long long)kXyNarrow * xy_cus() ||
         ((size_t)nx * ny * cellb < kXyCached &&
          xy_even<T>(nx, ny, Nv, kb, 4) > 1.2 * xy_even<T>(nx, ny, Nv, kb, xy_cols<T>()))))
        return launch_pfc_xy_cols<T, 4>(fin, fout, nx, ny, nvx, nvy, nvz, vx_lo, dvx, tau_dx, vy_lo, dvy, tau_dy, per,
                                        finf, sink, st);
    if (cellb >= 65536)
        return launch_pfc_xy_cols<T, xy_cols_big<T>()>(fin, fout, nx, ny, nvx, nvy, nvz, vx_lo, dvx, tau_dx, vy_lo, dvy, tau_dy,
                                             per, finf, sink, st);
    return launch_pfc_xy_cols<T, xy_cols<T>()>(fin, fout, nx, ny, nvx, nvy, nvz, vx_lo, dvx, tau_dx, vy_lo, dvy,
                                               tau_dy, per, finf, sink, st);
}

template <class T>
hipError_t launch_pfc_v1(const T* fin, T* fout, int nx, int nv, double* E, const double* mom, const double* g,
                         double q, double qm_tau_dv, MaxRef finf, const MaxSink& sink, hipStream_t st) {
    const int threads = nv >= 256 ? 256 : ((nv + 63) / 64) * 64;
    const size_t shm = sizeof(T) * (size_t)(nv + 4);
    const LineField S{E, mom, g, q};
    hipLaunchKernelGGL((finf.n > 1 ? pfc_v1_kernel<T, true> : pfc_v1_kernel<T, false>), dim3(nx), dim3(threads), shm,
                       st, fin, fout, nx, nv, S, qm_tau_dv, finf, sink.target<T>(nx));
    return finish_max<T>(sink, nx, st);
}

size_t v3_shared_bytes(int nvx, int nvy, int nvz, size_t elem) {
    return elem * (size_t)nvx * nvy * (nvz | 1);
}

// Threads per block for a kernel whose blocks (one per cell) run n rounds over
// pens[0..n) pencils, one pencil per thread: the count that takes the least
// time if lane slots go through at a rate set by the waves resident on a CU
// (as many blocks as its LDS, its registers -- `cap` waves -- and the number of
// cells allow).  V, FP32, per call: 5000 cells of 20x16x24 373 us with 64
// threads, 244 with 128, 191 with 256 (the LDS holds five blocks); 200 such
// cells 117, 75, 58, and 36 with 512; 20000 cells of 10^3 101 with 64, 144 with
// 256 (100 pencils).  Ties go to more threads if `wide`, else to fewer.
int pencil_threads(const int* pens, int n, size_t lds, int cap, long long cells, bool wide) {
    const long long cus = xy_cus();
    long long held = 163840 / (lds + 256);
    const long long per_cu = (cells + cus - 1) / cus;
    if (per_cu < held) held = per_cu;
    int best = 64;
    double best_cost = 0.0;
    for (int t = 64; t <= 512; t *= 2) {
        const int w = t / 64;
        long long blocks = cap / w < held ? cap / w : held;
        if (blocks < 1) blocks = 1;
        long long slots = 0;
        for (int k = 0; k < n; ++k) slots += (long long)((pens[k] + t - 1) / t) * t;
        const double cost = (double)slots / (double)(blocks * w);
        if (t == 64 || cost < best_cost || (wide && cost == best_cost)) {
            best = t;
            best_cost = cost;
        }
    }
    return best;
}

template <class T>
hipError_t launch_pfc_v3(const T* fin, T* fout, long long cells, const double* E, const double* B,
                         const V3Params& P, MaxRef finf, const MaxSink& sink, hipStream_t st) {
    const int nmax = P.nvx > P.nvy ? (P.nvx > P.nvz ? P.nvx : P.nvz) : (P.nvy > P.nvz ? P.nvy : P.nvz);
    const size_t shm = v3_shared_bytes(P.nvx, P.nvy, P.nvz, sizeof(T));
    const bool cube = P.nvx == P.nvy && P.nvy == P.nvz;
    auto* mo = sink.target<T>(cells);
    const dim3 grid((unsigned)cells);
    if (cube && P.nvx == kBigCube) {
        // one cell per CU (its LDS); 578 threads = two v_x pencils each
        if constexpr (sizeof(T) == 4)
            hipLaunchKernelGGL((finf.n > 1 ? pfc_v3_cube_kernel<T, kBigCube, 578, true> : pfc_v3_cube_kernel<T, kBigCube, 578, false>), grid, dim3(578), 0, st, fin, fout, E, B, P,
                               finf, mo);
        else        // the FP64 block is twice the LDS: half its v_x planes at a time
            hipLaunchKernelGGL((finf.n > 1 ? pfc_v3_planes_kernel<T, kBigCube, 512, 17, true> : pfc_v3_planes_kernel<T, kBigCube, 512, 17, false>), grid, dim3(512), 0, st, fin, fout, E, B,
                               P, finf, mo);
        return finish_max<T>(sink, cells, st);
    }
    if (cube && P.nvx == 16) {
        hipLaunchKernelGGL((finf.n > 1 ? pfc_v3_cube_kernel<T, 16, 256, true> : pfc_v3_cube_kernel<T, 16, 256, false>), grid, dim3(256), 0, st, fin, fout, E, B, P, finf, mo);
    } else if (cube && P.nvx == 12) {
        hipLaunchKernelGGL((finf.n > 1 ? pfc_v3_cube_kernel<T, 12, 192, true> : pfc_v3_cube_kernel<T, 12, 192, false>), grid, dim3(192), 0, st, fin, fout, E, B, P, finf, mo);
    } else if (cube && P.nvx == 8) {
        hipLaunchKernelGGL((finf.n > 1 ? pfc_v3_cube_kernel<T, 8, 64, true> : pfc_v3_cube_kernel<T, 8, 64, false>), grid, dim3(64), 0, st, fin, fout, E, B, P, finf, mo);
    } else if (nmax <= 32) {
        const int pens[5] = {P.nvy * P.nvz, P.nvx * P.nvz, P.nvx * P.nvy, P.nvx * P.nvz, P.nvy * P.nvz};
        const int threads = nmax <= 8 ? 64 : pencil_threads(pens, 5, shm, sizeof(T) == 4 ? 16 : 8, cells, true);
        hipLaunchKernelGGL((nmax <= 8 ? pfc_v3_kernel<T, 8, 64> : pfc_v3_kernel<T, 32, 512>), grid, dim3(threads), shm,
                           st, fin, fout, E, B, P, finf, mo);
    } else {
        return hipErrorInvalidValue;
    }
    return finish_max<T>(sink, cells, st);
}

// V(tau) by the backsubstitution split (any grid with every axis <= 32, and
// the 34^3 cube in FP32, whose padded block, 158 KB, fills one CU's LDS).
template <class T>
hipError_t launch_pfc_v3b(const T* fin, T* fout, long long cells, const double* E, const double* B,
                          const V3Params& P, MaxRef finf, const MaxSink& sink, hipStream_t st) {
    const int nmax = P.nvx > P.nvy ? (P.nvx > P.nvz ? P.nvx : P.nvz) : (P.nvy > P.nvz ? P.nvy : P.nvz);
    const size_t shm = v3_shared_bytes(P.nvx, P.nvy, P.nvz, sizeof(T));
    auto* mo = sink.target<T>(cells);
    const dim3 grid((unsigned)cells);
    const bool cube = P.nvx == P.nvy && P.nvy == P.nvz;
    if (nmax > 32) {
        if constexpr (sizeof(T) == 4) {
            if (!cube || P.nvx != kBigCube || shm > 160 * 1024) return hipErrorInvalidValue;
            // one workgroup per CU (the block fills the LDS): 640 threads, two
            // pencils each per sweep (1156 per sweep)
            hipLaunchKernelGGL((finf.n > 1 ? pfc_v3b_kernel<T, kBigCube, kBigCube, 640, true> : pfc_v3b_kernel<T, kBigCube, kBigCube, 640, false>),
                               grid, dim3(640), shm, st, fin, fout, E, B, P, finf, mo);
            return finish_max<T>(sink, cells, st);
        } else {
            return hipErrorInvalidValue;
        }
    }
    const int pens[3] = {P.nvy * P.nvz, P.nvx * P.nvz, P.nvx * P.nvy};
    const int threads = nmax <= 8 ? 64 : pencil_threads(pens, 3, shm, sizeof(T) == 4 ? 16 : 8, cells, true);
#define VL_V3B(N, L, NTH)                                                                                    \
    hipLaunchKernelGGL((finf.n > 1 ? pfc_v3b_kernel<T, N, L, NTH, true> : pfc_v3b_kernel<T, N, L, NTH, false>), grid, \
                       dim3(threads), shm, st, fin, fout, E, B, P, finf, mo)
    if (cube && P.nvx == 16)
        VL_V3B(16, 16, 512);
    else if (cube && P.nvx == 12)
        VL_V3B(12, 12, 512);
    else if (cube && P.nvx == 8)
        VL_V3B(8, 8, 64);
    else if (nmax <= 8)
        VL_V3B(0, 8, 64);
    else
        VL_V3B(0, 32, 512);
#undef VL_V3B
    return finish_max<T>(sink, cells, st);
}

template <class T>
hipError_t launch_array_max(const T* f, long long n, const MaxSink& sink, hipStream_t st) {
    long long blocks = (n + 2047) / 2048;
    if (blocks > kMaxArrayBlocks) blocks = kMaxArrayBlocks;
    if (blocks < 1) blocks = 1;
    const bool past = n * (long long)sizeof(T) > kLastLevelBytes;
    hipLaunchKernelGGL((past ? array_max_kernel<T, true> : array_max_kernel<T, false>), dim3((unsigned)blocks), dim3(256),
                       0, st, f, n, sink.target<T>(blocks));
    return finish_max<T>(sink, blocks, st);
}

#define VL_INST(T)                                                                                         \
    template hipError_t launch_pfc_x<T>(const T*, T*, int, int, long long, int, double, double, double,     \
                                        MaxRef, const MaxSink&, hipStream_t);                              \
    template hipError_t launch_pfc_v1<T>(const T*, T*, int, int, double*, const double*, const double*,      \
                                         double, double, MaxRef, const MaxSink&, hipStream_t);             \
    template hipError_t launch_pfc_v3<T>(const T*, T*, long long, const double*, const double*,             \
                                         const V3Params&, MaxRef, const MaxSink&, hipStream_t);            \
    template hipError_t launch_pfc_v3b<T>(const T*, T*, long long, const double*, const double*,            \
                                          const V3Params&, MaxRef, const MaxSink&, hipStream_t);           \
    template hipError_t launch_array_max<T>(const T*, long long, const MaxSink&, hipStream_t);              \
    template hipError_t launch_pfc_xy<T>(const T*, T*, int, int, int, int, int, double, double, double, double, \
                                         double, double, int, MaxRef, const MaxSink&, hipStream_t);        \
    template hipError_t launch_max_finalize<T>(const void*, long long, void*, hipStream_t);
VL_INST(float)
VL_INST(double)
#undef VL_INST

}  // namespace vl
