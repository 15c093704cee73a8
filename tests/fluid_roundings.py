"""The ten-moment fluid stage with every rounding of the kernels, on the host:
the oracle's formulas (oracle.fluid) in the operation order of
csrc/fluid_kernels.hip, with an exact fused multiply-add."""
import math

import numpy as np

EPS = 1e-6
A6, B6 = (0, 0, 0, 1, 1, 2), (0, 1, 2, 1, 2, 2)                              # P pairs
A9, B9, C9 = (0, 0, 0, 0, 0, 0, 1, 1, 1), (0, 0, 0, 1, 1, 2, 1, 1, 2), (0, 1, 2, 1, 2, 2, 1, 2, 2)
P_OF = np.array([[4, 5, 6], [5, 7, 8], [6, 8, 9]])
# component whose value is flux k, per direction; 10.. are the third moments of the P pairs
SRC = ((1, 4, 5, 6, 10, 11, 12, 13, 14, 15), (2, 5, 7, 8, 10, 11, 12, 13, 14, 15))
THIRD = ((0, 1, 2, 3, 4, 5), (1, 3, 4, 6, 7, 8))
PAR_U = np.array([1., 1., -1., 1., 1., -1., 1., 1., -1., 1.])
PAR_Q = np.array([1., -1., 1., 1., -1., 1., -1., 1., -1., 1.])


def _two_sum(a, b):
    s = a + b
    t = s - a
    return s, (a - (s - t)) + (b - t)


def fma(a, b, c):
    """Correctly rounded a b + c: the product exactly in two parts, the two
    low-order sums rounded to odd (Boldo and Melquiond, 2008)."""
    a, b, c = np.broadcast_arrays(*(np.asarray(x, dtype=np.float64) for x in (a, b, c)))
    p = a * b
    t = 134217729.0 * a
    ah = t - (t - a)
    al = a - ah
    t = 134217729.0 * b
    bh = t - (t - b)
    bl = b - bh
    e = ((ah * bh - p) + ah * bl + al * bh) + al * bl
    th, tl = _two_sum(c, e)
    vh, vl = _two_sum(p, th)
    z, r = _two_sum(tl, vl)
    bits = z.view(np.int64)
    step = np.where((r > 0) == (z > 0), 1, -1)
    odd = np.where((r != 0) & ((bits & 1) == 0), bits + step, bits).view(np.float64)
    return vh + odd


def cweno(a, b, c):
    dl, dr, d2, hc = b - a, c - b, fma(-2.0, b, c) + a, 0.5 * (c - a)
    el, er = fma(dl, dl, EPS), fma(dr, dr, EPS)
    ec = fma(hc, hc, fma(d2, d2 * (13.0 / 3.0), EPS))
    Dl, Dc, Dr = el * el, ec * ec, er * er
    tl, tc, tr = Dc * Dr, (Dl + Dl) * Dr, Dl * Dc
    inv = 1.0 / fma(Dl, Dc, fma(Dl + Dl, Dr, tl))
    wl, wc, wr = tl * inv, tc * inv, tr * inv
    side = fma(hc, wc, fma(dl, wl, dr * wr))
    even = d2 * (1.0 / 3.0)
    return fma(0.5, fma(even, wc, -side), b), fma(0.5, fma(even, wc, side), b)


def _speed(W, nu, pdd, m):
    u, mn = W[..., nu] / W[..., 0], m * W[..., 0]
    p = fma(-u, mn * u, W[..., pdd])
    return np.abs(u) + np.sqrt(np.maximum(3.0 * p / mn, 0.0))


def _ghosts(A, bc, par):
    """Two ghost rows (y) and columns (x) on every side."""
    ny, nx = A.shape[:2]
    j, i = np.arange(-2, ny + 2), np.arange(-2, nx + 2) % nx
    if bc == "periodic":
        return A[j % ny][:, i]
    src = np.where(j < 0, -1 - j, np.where(j >= ny, 2 * ny - 1 - j, j))
    out = A[src][:, i]
    out[(j < 0) | (j >= ny)] *= par
    return out


def third_moment(U, m, scale=None, y=None):
    """Qcal (nine components; zzz is not used) of zero heat flux, or of the
    network's, scale y."""
    u = [U[..., k] / U[..., 0] for k in (1, 2, 3)]
    mn2 = 2.0 * m * U[..., 0]
    Q = np.zeros(U.shape[:-1] + (10,))
    for k, (a, b, c) in enumerate(zip(A9, B9, C9)):
        first = u[b] * U[..., P_OF[a, c]]
        s = first + first if a == b else fma(u[a], U[..., P_OF[b, c]], first)
        s = fma(u[c], U[..., P_OF[a, b]], s)
        if y is not None:
            s = fma(scale, y[..., k].astype(np.float64), s)
        Q[..., k] = fma(-(mn2 * u[a] * u[b]), u[c], s)
    return Q


def gradient_source(Ug, n_inner, m, gchi, idx, idy):
    """Eq. 5's source of P from the state with ghosts."""
    n = Ug[..., 0]
    u = [Ug[..., k] / n for k in (1, 2, 3)]
    T = []
    for k, (a, b) in enumerate(zip(A6, B6)):
        mnu = m * n * u[a]
        T.append((Ug[..., 4 + k] - mnu * u[b] if k in (1, 4) else fma(-mnu, u[b], Ug[..., 4 + k])) / n)

    def at(t, dj, di):
        return t[2 + dj:t.shape[0] - 2 + dj, 2 + di:t.shape[1] - 2 + di]
    tr = at(T[0], 0, 0) + at(T[3], 0, 0) + at(T[5], 0, 0)
    g = gchi * (n_inner * np.sqrt(tr / (3.0 * m)))
    out = np.empty(n_inner.shape + (6,))
    for k, t in enumerate(T):
        lx = fma(-2.0, at(t, 0, 0), at(t, 0, 1)) + at(t, 0, -1)
        ly = fma(-2.0, at(t, 0, 0), at(t, 1, 0)) + at(t, -1, 0)
        out[..., k] = g * fma(lx, idx * idx, ly * (idy * idy))
    return out


def stage_3v(Us, Un, Qc, E, B, q, m, dx, dy, dt, a, b, bc, gchi=None):
    """U_out = a Un + b (Us + dt L(Us)); Qc [ny, nx, 10]."""
    idx, idy, im, qm = 1.0 / dx, 1.0 / dy, 1.0 / m, q / m
    Ug, Qg = _ghosts(Us, bc, PAR_U), _ghosts(Qc, bc, PAR_Q)
    diff = []
    for d in range(2):
        W = np.concatenate([Ug, Qg[..., THIRD[d]]], axis=-1)
        W = W[2:-2] if d == 0 else W[:, 2:-2].swapaxes(0, 1)      # sweep along axis 1
        lo, hi = cweno(W[:, :-2], W[:, 1:-1], W[:, 2:])
        nu, pdd = 1 + d, (4, 7)[d]
        Wm, Wp = hi[:, :-1], lo[:, 1:]
        ha = 0.5 * np.maximum(_speed(Wm, nu, pdd, m), _speed(Wp, nu, pdd, m))
        H = np.empty(Wm.shape[:-1] + (10,))
        for k in range(10):
            fm, fp = Wm[..., SRC[d][k]], Wp[..., SRC[d][k]]
            s = fma(im, fm, im * fp) if 1 <= k < 4 else fp + fm
            H[..., k] = fma(0.5, s, -(ha * (Wp[..., k] - Wm[..., k])))
        D = H[:, 1:] - H[:, :-1]
        diff.append(D if d == 0 else D.swapaxes(0, 1))
    u = [Us[..., k] for k in range(10)]
    Ev, Bv = [E[..., d] for d in range(3)], [B[..., d] for d in range(3)]
    S = [None,
         fma(-u[3], Bv[1], fma(Ev[0], u[0], Bv[2] * u[2])),
         fma(-u[1], Bv[2], fma(Ev[1], u[0], Bv[0] * u[3])),
         fma(-u[2], Bv[0], fma(Ev[2], u[0], Bv[1] * u[1]))]
    P = [[u[P_OF[i, j]] for j in range(3)] for i in range(3)]
    X = [[fma(-Bv[1], P[0][2], Bv[2] * P[0][1]) if r == 0 else fma(P[r][1], Bv[2], -(P[r][2] * Bv[1])),
          fma(P[r][2], Bv[0], -(P[r][0] * Bv[2])),
          fma(P[r][0], Bv[1], -(P[r][1] * Bv[0]))] for r in range(3)]
    for x, y in zip(A6, B6):
        nE = u[1 + y] * Ev[x]
        S.append(fma(q, nE + nE if x == y else fma(u[1 + x], Ev[y], nE), qm * (X[x][y] + X[y][x])))
    G = None if gchi is None else gradient_source(Ug, Us[..., 0], m, gchi, idx, idy)
    out = np.empty_like(Us)
    for k in range(10):
        d = fma(idx, diff[0][..., k], diff[1][..., k] * idy)
        L = -d if k == 0 else (fma(qm, S[k], -d) if k < 4 else S[k] - d)
        if G is not None and k >= 4:
            L = L + G[..., k - 4]
        s = fma(dt, L, u[k])
        out[..., k] = s if a == 0.0 else fma(b, s, a * Un[..., k])
    return out


def rk3_3v(U, third, fields, q, m, dx, dy, dt, bc, gchi=None):
    """One SSP-RK3 step; third(stage, state) gives Qcal, fields[stage] (E, B)."""
    cur = U
    for k, (a, b) in enumerate(((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0))):
        cur = stage_3v(cur, U, third(k, cur), *fields[k], q, m, dx, dy, dt, a, b, bc, gchi)
    return cur


def rk3_1v(U, Q, E, q, m, dx, dt):
    """One step of the 1V fluid, Q and E at the three stages."""
    cur = U
    ring = np.arange(-2, U.shape[0] + 2) % U.shape[0]
    for s, (a, b) in enumerate(((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0))):
        W = np.concatenate([cur, Q[s][:, None]], axis=-1)[ring]
        lo, hi = cweno(W[:-2], W[1:-1], W[2:])
        Wm, Wp = hi[:-1], lo[1:]
        wave = np.maximum(_speed(Wm, 1, 2, m), _speed(Wp, 1, 2, m))
        src = [np.zeros(len(cur)), (q / m) * cur[:, 0], 2.0 * q * cur[:, 1]]
        new = np.empty_like(cur)
        for k in range(3):
            f = [W_[:, k + 1] / m if k == 1 else W_[:, k + 1] for W_ in (Wp, Wm)]
            H = 0.5 * (f[0] + f[1]) - 0.5 * wave * (Wp[:, k] - Wm[:, k])
            v = fma(dt, fma(src[k], E[s], -((H[1:] - H[:-1]) / dx)), cur[:, k])
            new[:, k] = v if a == 0.0 else fma(b, v, a * U[:, k])
        cur = new
    return cur


def eq5_strength(q, m):
    """chi / k0 of Eq. 5."""
    return 2.0 * math.sqrt(2.0 / math.pi) * math.sqrt(m / (q * q))
