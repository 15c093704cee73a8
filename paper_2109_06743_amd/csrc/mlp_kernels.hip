// Learned heat-flux closure on gfx950: stencil features from the ten moments,
// a 64-64-64-64-16 tanh network evaluated and trained with BF16 MFMA
// (v_mfma_f32_16x16x16_bf16, FP32 accumulation), Adam on FP32 master
// weights, and the pieces the fluid update uses (third moment from the
// network, error of the network's heat flux against the kinetic one).
//
// Network layout (FP32 parameter vector, row-major [out][in]):
//   W1[64][64] b1[64] W2[64][64] b2[64] W3[64][64] b3[64] W4[16][64] b4[16]
// The network multiplies BF16-rounded weights and activations; biases,
// accumulation and tanh are FP32.
//
// Matrix products are computed transposed, H_l^T = W_l H_{l-1}^T, so that a
// 16x16 output tile of one layer (lane l holds rows 4(l/16)+j, column l%16)
// is already the B operand of the next layer (rows = the K index): samples
// run along the 16 lanes of a row group, features along (l/16, j), and no
// data moves between layers.
#include <type_traits>

#include "vl_internal.h"

namespace vl {
namespace {

constexpr int kIn = 64, kWid = 64, kOutPad = 16, kOut = 10;
constexpr int kOffW1 = 0, kOffB1 = 4096, kOffW2 = 4160, kOffB2 = 8256, kOffW3 = 8320, kOffB3 = 12416,
              kOffW4 = 12480, kOffB4 = 13504, kNParam = 13520;
constexpr int kLdw = 68;    // bf16 row stride of weight tiles in LDS (136 B rows keep 8-byte alignment)
constexpr int kLdt4 = 20;   // row stride of W4^T [64][16]
constexpr int kLds = 20;    // row stride of the per-wave transpose staging tiles [16][16]
constexpr int kPartStride = 13536;   // floats per block partial: gradient (13520) + loss, padded

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short bf16_of(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);     // round to nearest, ties to even
    return (unsigned short)(u >> 16);
}

__device__ __forceinline__ bf16x4 pack4(const f32x4& v) {
    bf16x4 r;
    r[0] = (short)bf16_of(v[0]);
    r[1] = (short)bf16_of(v[1]);
    r[2] = (short)bf16_of(v[2]);
    r[3] = (short)bf16_of(v[3]);
    return r;
}

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x4 lds4(const unsigned short* p) { return *reinterpret_cast<const bf16x4*>(p); }

// Weights of the network in LDS as BF16 (plus FP32 biases); the transposed
// copies are for the backward products.
struct NetLds {
    unsigned short w[3][kWid * kLdw];     // W1..W3 [out][in]
    unsigned short w4[kOutPad * kLdw];    // W4 [16][64]
    float bias[3 * kWid + kOutPad];
};
struct NetLdsT {
    unsigned short wt[2][kWid * kLdw];    // W2^T, W3^T [in][out]
    unsigned short wt4[kWid * kLdt4];     // W4^T [64][16]
};

__device__ __forceinline__ void load_net(const float* __restrict__ P, NetLds& N, NetLdsT* T) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    if (nthr == 512 && !((uintptr_t)P & 15u)) {
        // 512 threads, 16-byte aligned parameters: all seven float4 loads of a
        // thread are issued before the first conversion
        float4 v[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int e = i * 512 + tid;                      // float4 index over W1, W2, W3, W4
            const int off = e < 1024 ? kOffW1 : (e < 2048 ? kOffW2 : (e < 3072 ? kOffW3 : kOffW4));
            v[i] = e < 3072 + 256 ? reinterpret_cast<const float4*>(P + off)[e & 1023] : float4{0.f, 0.f, 0.f, 0.f};
        }
        const float bv = tid < 3 * kWid + kOutPad
                             ? P[tid < 64 ? kOffB1 + tid
                                          : (tid < 128 ? kOffB2 + tid - 64
                                                       : (tid < 192 ? kOffB3 + tid - 128 : kOffB4 + tid - 192))]
                             : 0.f;
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int e = i * 512 + tid;
            if (e >= 3072 + 256) continue;
            const int w = 4 * (e & 1023), r = w / kIn, c = w % kIn;
            const unsigned short h[4] = {bf16_of(v[i].x), bf16_of(v[i].y), bf16_of(v[i].z), bf16_of(v[i].w)};
            const uint2 pk = {(unsigned)h[0] | ((unsigned)h[1] << 16), (unsigned)h[2] | ((unsigned)h[3] << 16)};
            *reinterpret_cast<uint2*>(e < 3072 ? &N.w[e >> 10][r * kLdw + c] : &N.w4[r * kLdw + c]) = pk;
            if (T && i >= 2) {                            // i = 0, 1: W1
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (i < 6) T->wt[(i - 2) / 2][(c + k) * kLdw + r] = h[k];
                    else T->wt4[(c + k) * kLdt4 + r] = h[k];
                }
            }
        }
        if (tid < 3 * kWid + kOutPad) N.bias[tid] = bv;
        return;
    }
    if (nthr == 256 && !T && !((uintptr_t)P & 15u)) {
        // 256 threads (no transposes): 13 float4 loads each
        float4 v[13];
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            const int off = i < 4 ? kOffW1 : (i < 8 ? kOffW2 : kOffW3);
            v[i] = reinterpret_cast<const float4*>(P + off)[(i & 3) * 256 + tid];
        }
        v[12] = reinterpret_cast<const float4*>(P + kOffW4)[tid];
        const float bv = tid < 3 * kWid + kOutPad
                             ? P[tid < 64 ? kOffB1 + tid
                                          : (tid < 128 ? kOffB2 + tid - 64
                                                       : (tid < 192 ? kOffB3 + tid - 128 : kOffB4 + tid - 192))]
                             : 0.f;
#pragma unroll
        for (int i = 0; i < 13; ++i) {
            const int e = 4 * ((i & 3) * 256 + tid);          // first of 4 consecutive inputs of one row
            const int r = e / kIn, c = e % kIn;
            const unsigned short h[4] = {bf16_of(v[i].x), bf16_of(v[i].y), bf16_of(v[i].z), bf16_of(v[i].w)};
            const uint2 pk = {(unsigned)h[0] | ((unsigned)h[1] << 16), (unsigned)h[2] | ((unsigned)h[3] << 16)};
            if (i < 12) {
                const int l = i / 4;
                *reinterpret_cast<uint2*>(&N.w[l][r * kLdw + c]) = pk;
            } else {
                const int r4 = 4 * tid / kWid, c4 = 4 * tid % kWid;
                *reinterpret_cast<uint2*>(&N.w4[r4 * kLdw + c4]) = pk;
            }
        }
        if (tid < 3 * kWid + kOutPad) N.bias[tid] = bv;
        return;
    }
    for (int e = tid; e < 3 * kWid * kIn; e += nthr) {
        const int l = e / (kWid * kIn), r = (e / kIn) % kWid, c = e % kIn;
        const int off = l == 0 ? kOffW1 : (l == 1 ? kOffW2 : kOffW3);
        const unsigned short v = bf16_of(P[off + r * kIn + c]);
        N.w[l][r * kLdw + c] = v;
        if (T && l > 0) T->wt[l - 1][c * kLdw + r] = v;
    }
    for (int e = tid; e < kOutPad * kWid; e += nthr) {
        const int r = e / kWid, c = e % kWid;
        const unsigned short v = bf16_of(P[kOffW4 + e]);
        N.w4[r * kLdw + c] = v;
        if (T) T->wt4[c * kLdt4 + r] = v;
    }
    for (int e = tid; e < 3 * kWid + kOutPad; e += nthr) {
        const int off = e < 64 ? kOffB1 + e : (e < 128 ? kOffB2 + e - 64 : (e < 192 ? kOffB3 + e - 128 : kOffB4 + e - 192));
        N.bias[e] = P[off];
    }
}

// tanh through the exponential, tanh|x| = 1 - 2 / (exp(2|x|) + 1), with the
// sign put back: absolute error below 1e-7, far under the BF16 rounding the
// activations then take; exp(2|x|) = inf gives exactly 1.
__device__ __forceinline__ float tanh_exp(float x) {
    const float e = __expf(2.f * fabsf(x));
    return copysignf(1.f - 2.f * __builtin_amdgcn_rcpf(e + 1.f), x);
}

// Forward pass of one 16-sample tile by one wave.  hb[0] = features, hb[1..3]
// = hidden activations (BF16 operands), h[0..2] = the same in FP32 (for tanh'),
// y = outputs (rows 4g+j of the 16 outputs, sample s).
struct Tile {
    bf16x4 hb[4][4];
    f32x4 h[3][4];
    f32x4 y;
};

// Source row of batch row r: idx[r] (rows outside [0, nrows) count as
// padding, -1) or r itself; -1 past the batch.
__device__ __forceinline__ long long source_row(long long r, long long n, const long long* __restrict__ idx,
                                                long long nrows) {
    if (r >= n) return -1;
    if (!idx) return r;
    const long long q = idx[r];
    return (q >= 0 && q < nrows) ? q : -1;
}

// This lane's features (sample s, inputs 16kb+4g..16kb+4g+3) of source row
// `row`; zeros for row -1.
__device__ __forceinline__ void load_features(const unsigned short* __restrict__ x, long long row, uint2 (&v)[4]) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
        v[kb] = row >= 0 ? *reinterpret_cast<const uint2*>(x + row * kIn + 16 * kb + 4 * g) : uint2{0u, 0u};
}

__device__ __forceinline__ void forward_from(const uint2 (&xv)[4], const NetLds& N, Tile& T) {
    const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) T.hb[0][kb] = *reinterpret_cast<const bf16x4*>(&xv[kb]);
#pragma unroll
    for (int L = 0; L < 3; ++L) {
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            const float* b = N.bias + L * kWid + 16 * ob + 4 * g;
            f32x4 acc = {b[0], b[1], b[2], b[3]};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                acc = mfma16(lds4(N.w[L] + (16 * ob + s) * kLdw + 16 * kb + 4 * g), T.hb[L][kb], acc);
            f32x4 h;
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = tanh_exp(acc[j]);
            T.hb[L + 1][ob] = pack4(h);
        }
    }
    const float* b4 = N.bias + 3 * kWid + 4 * g;
    f32x4 acc = {b4[0], b4[1], b4[2], b4[3]};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) acc = mfma16(lds4(N.w4 + s * kLdw + 16 * kb + 4 * g), T.hb[3][kb], acc);
    T.y = acc;
}

__device__ __forceinline__ void forward_tile(const unsigned short* __restrict__ x, long long n, long long tile,
                                             const NetLds& N, Tile& T) {
    uint2 v[4];
    load_features(x, source_row(tile * 16 + (threadIdx.x & 15), n, nullptr, 0), v);
    forward_from(v, N, T);
}

// Tile `ob` of a layer held in output layout (lane: rows 4g+j, column s = the
// sample) into LDS by features, stage[row][sample], where row s, samples 4g+j
// can be read as the operand of a product over samples; or by samples,
// ex[sample][row], which is the B operand of the next layer.
__device__ __forceinline__ void put_by_feature(unsigned short* stage, int ob, const bf16x4& v) {
    const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) stage[(16 * ob + 4 * g + j) * kLds + s] = (unsigned short)v[j];
}
__device__ __forceinline__ void put_by_sample(unsigned short* ex, int ob, const bf16x4& v) {
    const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
    *reinterpret_cast<bf16x4*>(ex + s * kLdw + 16 * ob + 4 * g) = v;
}
__device__ __forceinline__ void get_by_sample(const unsigned short* ex, bf16x4 (&v)[4]) {
    const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) v[kb] = lds4(ex + s * kLdw + 16 * kb + 4 * g);
}

__device__ __forceinline__ float sum16(float v) {
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 8, 64);
    return v;
}

}  // namespace

// --------------------------------------------------------------- features --
// Per cell: n, u, T (6) of the centre and its 8 neighbours (x periodic, y
// mirrored with u_y, T_xy, T_yz negated), the species and the direction of
// the cell-centred magnetic field -> 64 features rounded FP64 -> FP32 ->
// BF16, and the scale n m v_t^3.
__device__ __forceinline__ bool local_nuT(const double* __restrict__ M, int stride, long long c, double m,
                                          bool mir, double& n, double (&u)[3], double (&T)[6]) {
    n = M[c * stride];
    const double inv = 1.0 / n;
    u[0] = M[c * stride + 1] * inv;
    u[1] = M[c * stride + 2] * inv;
    u[2] = M[c * stride + 3] * inv;
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int k = 0; k < 6; ++k) T[k] = (M[c * stride + 4 + k] - m * n * u[pa[k]] * u[pb[k]]) * inv;
    if (mir) {
        u[1] = -u[1];
        T[1] = -T[1];
        T[4] = -T[4];
    }
    return true;
}

// Species blockIdx.z of the set (species index s0 + blockIdx.z); its
// features, outputs and scales are stored after those of the set's earlier
// species.  A 512-thread block covers 4 rows x 64 columns of cells: n, u, T of
// its 6 x 66 stencil cells are formed once each into LDS (rather than nine
// times, once per neighbour), two threads then form each cell's features (34
// and 30 of them) from there as packed BF16 rows in LDS.  kNet = false: the
// rows leave for x, every wave store writing 256 contiguous bytes.  kNet: the
// block's waves run the network on them, two 16-cell tiles each, and only the
// outputs leave: the rows need not go through memory (2 x 128 B a cell) and a
// launch goes.  256 x 128 cells, two species: 15.7 us for the features by one
// thread per cell and 12.0 for the network, 15.2 in one.
constexpr int kFeatCols = 64, kFeatRows = 4, kFeatCells = kFeatCols * kFeatRows;
union FeatLds {
    double nut[kFeatRows + 2][kFeatCols + 2][11];   // n, u, T (padded against bank conflicts)
    unsigned out[kFeatCells][34];                    // packed BF16 feature rows (padded, 8-byte aligned)
};
struct NoNet {};

template <bool kNet>
__global__ void __launch_bounds__(2 * kFeatCells)
mlp_features_kernel(MlpSet S, int s0, int stride, const double* __restrict__ B, int nx, int ny,
                    unsigned short* __restrict__ x, double* __restrict__ scale, const float* __restrict__ P,
                    float* __restrict__ y) {
    __shared__ FeatLds L;
    __shared__ typename std::conditional<kNet, NetLds, NoNet>::type N;
    const int sp = blockIdx.z;
    const double* __restrict__ M = S.M[sp];
    const double m = S.m[sp];
    const int species = s0 + sp;
    if constexpr (kNet) {
        y += (size_t)sp * nx * ny * kOutPad;
        load_net(P, N, nullptr);
    } else {
        x += (size_t)sp * nx * ny * kIn;
    }
    scale += (size_t)sp * nx * ny;
    const int i0 = blockIdx.x * kFeatCols, j0 = blockIdx.y * kFeatRows;
    const int tid = threadIdx.x;
    for (int q = tid; q < (kFeatRows + 2) * (kFeatCols + 2); q += 2 * kFeatCells) {
        const int rr = q / (kFeatCols + 2), cc = q % (kFeatCols + 2);
        double* d = L.nut[rr][cc];
        int jj = j0 - 1 + rr;
        if (jj > ny) {             // below the mirror of row ny-1: feeds no cell
#pragma unroll
            for (int k = 0; k < 10; ++k) d[k] = 0.0;
            continue;
        }
        bool mir = false;
        if (jj < 0) { jj = -1 - jj; mir = true; }
        if (jj >= ny) { jj = 2 * ny - 1 - jj; mir = true; }
        const int ii = ((i0 - 1 + cc) % nx + nx) % nx;
        double nn, uu[3], TT[6];
        local_nuT(M, stride, (long long)jj * nx + ii, m, mir, nn, uu, TT);
        d[0] = nn;
#pragma unroll
        for (int k = 0; k < 3; ++k) d[1 + k] = uu[k];
#pragma unroll
        for (int k = 0; k < 6; ++k) d[4 + k] = TT[k];
    }
    __syncthreads();
    const bool second = tid >= kFeatCells;         // wave-uniform: which part of the features
    const int ct = tid & (kFeatCells - 1);
    const int r = ct / kFeatCols, cl = ct % kFeatCols;
    const int i = i0 + cl, j = j0 + r;
    const bool valid = i < nx && j < ny;
    float f[34];    // features are rounded to FP32 (then BF16) anyway
#pragma unroll
    for (int k = 0; k < 34; ++k) f[k] = 0.f;
    double sc = 0.0;
    if (valid) {
        const double* C = L.nut[r + 1][cl + 1];
        const double n0 = C[0];
        const double Tref = (C[4] + C[7] + C[9]) / 3.0;
        if (n0 > 1e-12 && Tref > 0.0) {
            const double vt = sqrt(Tref / m);
            const double ivt = 1.0 / vt, iT = 1.0 / Tref, in0 = 1.0 / n0;
            sc = n0 * m * vt * vt * vt;
            // five stencil fields n/n_c, u/v_t, T/T_ref at offset (dj, di)
            auto differences = [&](int k0, float* out) {
#pragma unroll
                for (int q = 0; q < 5; ++q) {
                    const int k = k0 + q;
                    const double sk = k == 0 ? in0 : (k < 4 ? ivt : iT);
                    auto P = [&](int dj, int di) { return L.nut[r + 1 + dj][cl + 1 + di][k] * sk; };
                    const double c0 = P(0, 0);
                    out[5 * q + 0] = (float)((P(0, 1) - P(0, -1)) / 2.0);
                    out[5 * q + 1] = (float)((P(1, 0) - P(-1, 0)) / 2.0);
                    out[5 * q + 2] = (float)(P(0, 1) - 2.0 * c0 + P(0, -1));
                    out[5 * q + 3] = (float)(P(1, 0) - 2.0 * c0 + P(-1, 0));
                    out[5 * q + 4] = (float)((P(1, 1) - P(-1, 1) - P(1, -1) + P(-1, -1)) / 4.0);
                }
            };
            if (!second) {         // features 0 .. 33
                f[0] = (float)(C[1] * ivt);
                f[1] = (float)(C[2] * ivt);
                f[2] = (float)(C[3] * ivt);
#pragma unroll
                for (int k = 0; k < 6; ++k) f[3 + k] = (float)(C[4 + k] * iT);
                differences(0, f + 9);
            } else {               // features 34 .. 63
                differences(5, f);
                if (species == 0) f[25] = 1.f;
                else f[26] = 1.f;
                if (B) {     // direction of the cell-centred magnetic field
                    const long long c = (long long)j * nx + i;
                    const double bx = B[c * 3], by = B[c * 3 + 1], bz = B[c * 3 + 2];
                    const double bn = sqrt(bx * bx + by * by + bz * bz);
                    if (bn > 1e-12) {
                        f[27] = (float)(bx / bn);
                        f[28] = (float)(by / bn);
                        f[29] = (float)(bz / bn);
                    }
                }
            }
        }
    }
    __syncthreads();     // every read of the stencil values is done: the union now holds the output
    auto pack = [&](int k) { return bf16_of(f[2 * k]) | ((unsigned)bf16_of(f[2 * k + 1]) << 16); };
    if (!second) {
#pragma unroll
        for (int k = 0; k < 17; ++k) L.out[ct][k] = pack(k);
        if (valid) scale[(long long)j * nx + i] = sc;
    } else {
#pragma unroll
        for (int k = 0; k < 15; ++k) L.out[ct][17 + k] = pack(k);
    }
    __syncthreads();
    if constexpr (kNet) {
        const int lane = tid & 63, s = lane & 15, g = lane >> 4;
#pragma unroll 1
        for (int t = tid / 64; t < kFeatCells / 16; t += 2 * kFeatCells / 64) {
            const int cell = t * 16 + s;
            uint2 v[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) v[kb] = *reinterpret_cast<const uint2*>(&L.out[cell][8 * kb + 2 * g]);
            Tile T;
            forward_from(v, N, T);
            const int ii = i0 + cell % kFeatCols, jj = j0 + cell / kFeatCols;
            if (ii < nx && jj < ny) *reinterpret_cast<f32x4*>(y + ((long long)jj * nx + ii) * kOutPad + 4 * g) = T.y;
        }
    } else {
        for (int q = tid; q < kFeatCells * 32; q += 2 * kFeatCells) {
            const int rr = q >> 5, part = q & 31;
            const int ii = i0 + rr % kFeatCols, jj = j0 + rr / kFeatCols;
            if (ii < nx && jj < ny)
                reinterpret_cast<unsigned*>(x + ((long long)jj * nx + ii) * kIn)[part] = L.out[rr][part];
        }
    }
}

// Heat-flux tensor of one cell from its raw moments (TRIPLES order).
__device__ __forceinline__ void heat_flux_cell(const double* __restrict__ M, long long c, double m, double (&Q)[10],
                                               double& n, double (&u)[3], double& Tref) {
    n = M[c * 20];
    const double inv = 1.0 / n;
    u[0] = M[c * 20 + 1] * inv;
    u[1] = M[c * 20 + 2] * inv;
    u[2] = M[c * 20 + 3] * inv;
    double P[3][3];
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int k = 0; k < 6; ++k) P[pa[k]][pb[k]] = P[pb[k]][pa[k]] = M[c * 20 + 4 + k];
    Tref = ((P[0][0] - m * n * u[0] * u[0]) + (P[1][1] - m * n * u[1] * u[1]) + (P[2][2] - m * n * u[2] * u[2])) *
           inv / 3.0;
    const int ta[10] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 2}, tb[10] = {0, 0, 0, 1, 1, 2, 1, 1, 2, 2},
              tc[10] = {0, 1, 2, 1, 2, 2, 1, 2, 2, 2};
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        const int a = ta[k], b = tb[k], d = tc[k];
        Q[k] = M[c * 20 + 10 + k] - (u[a] * P[b][d] + u[b] * P[a][d] + u[d] * P[a][b]) +
               2.0 * m * n * u[a] * u[b] * u[d];
    }
}

__global__ void mlp_targets_kernel(const double* __restrict__ M, long long cells, double m, float* __restrict__ y) {
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells) return;
    double Q[10], n, u[3], Tref;
    heat_flux_cell(M, c, m, Q, n, u, Tref);
    const bool ok = n > 1e-12 && Tref > 0.0;
    const double vt = ok ? sqrt(Tref / m) : 1.0;
    const double inv = ok ? 1.0 / (n * m * vt * vt * vt) : 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) y[c * 16 + k] = k < kOut ? (float)(Q[k < kOut ? k : 0] * inv) : 0.0f;
}

// ---------------------------------------------------------------- forward --
__global__ void __launch_bounds__(256)
mlp_forward_kernel(const float* __restrict__ P, const unsigned short* __restrict__ x, long long n,
                   float* __restrict__ y) {
    __shared__ NetLds N;
    load_net(P, N, nullptr);
    __syncthreads();
    const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
    const long long tiles = (n + 15) / 16;
    const long long nw = (long long)gridDim.x * (blockDim.x / 64);
    for (long long t = (long long)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; t < tiles; t += nw) {
        Tile T;
        forward_tile(x, n, t, N, T);
        const long long row = t * 16 + s;
        if (row < n) *reinterpret_cast<f32x4*>(y + row * 16 + 4 * g) = T.y;
    }
}

// --------------------------------------------------------------- gradient --
// Block b handles tiles [t0, t1), four at a time.  Two waves share a tile: each
// computes half of every layer's units, forward and backward, and they exchange
// the halves through LDS (by samples, two buffers in turn); they also leave the
// BF16 activations h and pre-activation gradients dA by features.  Then waves
// 2l, 2l+1 accumulate the weight gradient of layer l+1 over the four tiles, half
// of its rows (layer 4: columns) each, in MFMA accumulators kept over the
// block's tiles; biases are summed in FP32 from dA before its rounding, in the
// order of the tiles too, so the sums do not depend on how tiles are shared out.
// Each
// block writes one partial gradient and no floating-point atomics are used (the
// sum over blocks is done in a fixed order).
//
// A wave alone on its SIMD takes a tile's 52 + 36 products, 192 tanh and their
// packing in sequence, so the time is the longest wave's chain: at 16384 rows
// (four tiles a block) 18.5 us; 31 when every wave computed every tile for itself
// and kept one layer's gradient.
constexpr int kTilesIn = 4;
struct TileLds {
    unsigned short h[4][kWid * kLds];      // features and hidden activations, by features
    unsigned short d[3][kWid * kLds];      // dA1..dA3, by features
    unsigned short dy[kOutPad * kLds];
    unsigned short ex[2][16 * kLdw];
};

__global__ void __launch_bounds__(512)
mlp_grad_kernel(const float* __restrict__ P, const unsigned short* __restrict__ x, const float* __restrict__ t,
                long long n, long long tiles_per_block, float inv_norm, float* __restrict__ part,
                const long long* __restrict__ idx, long long nrows) {
    __shared__ NetLds N;
    __shared__ NetLdsT NT;
    __shared__ TileLds TL[kTilesIn];
    __shared__ f32x4 bsum[13][64];                 // bias sums, [4 layer + tile of 16 rows][lane]
    __shared__ float lred[kTilesIn];
    const int w = threadIdx.x / 64, lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
    const int q = w >> 1, p = w & 1;               // tile of the four; half of the units
    const int l = q;                               // layer - 1 whose gradient this wave keeps
    TileLds& X = TL[q];
    const long long tiles = (n + 15) / 16;
    const long long t0 = (long long)blockIdx.x * tiles_per_block;
    const long long t1 = t0 + tiles_per_block < tiles ? t0 + tiles_per_block : tiles;
    auto row_at = [&](long long tile) -> long long {
        return tile < t1 ? source_row(tile * 16 + s, n, idx, nrows) : -1;
    };
    // the features and targets of the next tile and the source row of the one
    // after are loaded while this tile is computed
    long long r1 = row_at(t0 + q);
    load_net(P, N, &NT);
    uint2 xv[4];
    f32x4 tv = {0.f, 0.f, 0.f, 0.f};
    load_features(x, r1, xv);
    if (r1 >= 0) tv = *reinterpret_cast<const f32x4*>(t + r1 * 16 + 4 * g);
    long long r2 = row_at(t0 + q + kTilesIn);
    f32x4 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int e = w; e < 13; e += 8) bsum[e][lane] = f32x4{0.f, 0.f, 0.f, 0.f};
    float lsum = 0.f;
    __syncthreads();
    for (long long base = t0; base < t1; base += kTilesIn) {
        const bool live = base + q < t1;           // the same for both waves of a tile
        const long long row = r1;
        bf16x4 in[4];                              // operand of the next product: all 64 rows, this sample
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) in[kb] = *reinterpret_cast<const bf16x4*>(&xv[kb]);
        const f32x4 tt = tv;
        r1 = r2;
        load_features(x, r1, xv);
        if (r1 >= 0) tv = *reinterpret_cast<const f32x4*>(t + r1 * 16 + 4 * g);
        r2 = row_at(base + q + 2 * kTilesIn);
        f32x4 h[3][2], dA[3][2], dy = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int L = 0; L < 3; ++L) {
            if (live) {
                if (L == 0) {
                    put_by_feature(X.h[0], 2 * p, p ? in[2] : in[0]);
                    put_by_feature(X.h[0], 2 * p + 1, p ? in[3] : in[1]);
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int ob = 2 * p + u;
                    const float* b = N.bias + L * kWid + 16 * ob + 4 * g;
                    f32x4 a = {b[0], b[1], b[2], b[3]};
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb)
                        a = mfma16(lds4(N.w[L] + (16 * ob + s) * kLdw + 16 * kb + 4 * g), in[kb], a);
#pragma unroll
                    for (int j = 0; j < 4; ++j) h[L][u][j] = tanh_exp(a[j]);
                    const bf16x4 hb = pack4(h[L][u]);
                    put_by_sample(X.ex[L & 1], ob, hb);
                    put_by_feature(X.h[L + 1], ob, hb);
                }
            }
            __syncthreads();
            if (live) get_by_sample(X.ex[L & 1], in);
        }
        // the outputs (both waves), dY and dA3 = (W4^T dY) * (1 - h3^2)
        auto put_dA = [&](int L, int u, const f32x4& d, unsigned short* ex) {
#pragma unroll
            for (int j = 0; j < 4; ++j) dA[L][u][j] = d[j] * (1.f - h[L][u][j] * h[L][u][j]);
            const bf16x4 b = pack4(dA[L][u]);
            put_by_feature(X.d[L], 2 * p + u, b);
            if (ex) put_by_sample(ex, 2 * p + u, b);
        };
        if (live) {
            const float* b4 = N.bias + 3 * kWid + 4 * g;
            f32x4 y = {b4[0], b4[1], b4[2], b4[3]};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) y = mfma16(lds4(N.w4 + s * kLdw + 16 * kb + 4 * g), in[kb], y);
            if (row >= 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d = (4 * g + j < kOut) ? y[j] - tt[j] : 0.f;
                    lsum += d * d;
                    dy[j] = 2.f * d * inv_norm;
                }
            }
            const bf16x4 dyb = pack4(dy);
            if (p == 0) put_by_feature(X.dy, 0, dyb);
#pragma unroll
            for (int u = 0; u < 2; ++u)
                put_dA(2, u, mfma16(lds4(NT.wt4 + (16 * (2 * p + u) + s) * kLdt4 + 4 * g), dyb, f32x4{0.f, 0.f, 0.f, 0.f}),
                       X.ex[1]);
        }
        // dA2, dA1: (W_{L+1}^T dA) * (1 - h_L^2)
#pragma unroll
        for (int L = 1; L >= 0; --L) {
            __syncthreads();
            if (!live) continue;
            get_by_sample(X.ex[L], in);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
                    d = mfma16(lds4(NT.wt[L] + (16 * (2 * p + u) + s) * kLdw + 16 * kb + 4 * g), in[kb], d);
                put_dA(L, u, d, L ? X.ex[0] : nullptr);
            }
        }
        __syncthreads();
        // weight gradients dW = dA h^T (dY h3^T) tile by tile; beside each, the
        // waves of that tile add to the bias sums
        for (int k = 0; k < kTilesIn && base + k < t1; ++k) {
            if (k == q) {
#pragma unroll
                for (int L = 0; L < 3; ++L)
#pragma unroll
                    for (int u = 0; u < 2; ++u) bsum[4 * L + 2 * p + u][lane] += dA[L][u];
                if (p == 0) bsum[12][lane] += dy;
            }
            const TileLds& Y = TL[k];
            if (l == 3) {
                const bf16x4 a = lds4(Y.dy + s * kLds + 4 * g);
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[0][u] = mfma16(a, lds4(Y.h[3] + (16 * (2 * p + u) + s) * kLds + 4 * g), acc[0][u]);
            } else {
                bf16x4 hT[4];
#pragma unroll
                for (int ib = 0; ib < 4; ++ib) hT[ib] = lds4(Y.h[l] + (16 * ib + s) * kLds + 4 * g);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bf16x4 a = lds4(Y.d[l] + (16 * (2 * p + u) + s) * kLds + 4 * g);
#pragma unroll
                    for (int ib = 0; ib < 4; ++ib) acc[u][ib] = mfma16(a, hT[ib], acc[u][ib]);
                }
            }
            __syncthreads();
        }
    }
    // this block's partial gradient
    float* out = part + (long long)blockIdx.x * kPartStride;
    if (l == 3) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) out[kOffW4 + (4 * g + j) * kWid + 16 * (2 * p + u) + s] = acc[0][u][j];
    } else {
        float* o = out + (l == 0 ? kOffW1 : (l == 1 ? kOffW2 : kOffW3));
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o[(16 * (2 * p + u) + 4 * g + j) * kWid + 16 * ib + s] = acc[u][ib][j];
    }
    for (int e = w; e < 13; e += 8) {
        const f32x4 d = bsum[e][lane];
        float* o = out + (e < 4 ? kOffB1 : (e < 8 ? kOffB2 : (e < 12 ? kOffB3 : kOffB4))) + 16 * (e & 3) + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float v = sum16(d[j]);
            if (s == 0) o[j] = v;
        }
    }
    if (p == 0) {
        float v = lsum;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) lred[q] = v * inv_norm;
    }
    __syncthreads();
    if (threadIdx.x == 0) out[kNParam] = (lred[0] + lred[1]) + (lred[2] + lred[3]);
}

// One Adam update (optional, after the gradient sum).
struct AdamArgs {
    float* P;          // null: no update
    float* m1;
    float* m2;
    float lr, beta1, beta2, eps, bc1, bc2;
};

// Sum of the block partials: grad[0..13519], loss at [13520].  Block i covers
// entries 64i..64i+63.  Partials form 16 chains, j, j + 16, j + 32, ..., each
// added up in order by one wave, all of a full launch's sixteen loads in flight;
// chain totals are added as ((j, j+4), (j+8, j+12)) for j = 0..3 and then over
// j.  Of a launch with fewer than 256 partials, what remains of j, j + 4, j + 8,
// ... past the last whole 64 goes to chain j (j < 4).  A fixed order, the same on
// every call.  With A.P set, the Adam update of the same entries follows.  256
// partials (13.8 MB): 7.4 us with four waves a block, 4.6 with sixteen.
__global__ void __launch_bounds__(1024)
mlp_reduce_kernel(const float* __restrict__ part, int nblocks, float* __restrict__ grad, AdamArgs A) {
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    const bool mine = w == 0 && A.P && p < kNParam;
    float m1 = 0.f, m2 = 0.f, P0 = 0.f;
    if (mine) {
        m1 = A.m1[p];
        m2 = A.m2[p];
        P0 = A.P[p];
    }
    float acc = 0.f;
    if (p <= kNParam) {
        const float* __restrict__ src = part + p;
        // whole rounds of 64 partials that j = w & 3 takes part in: j + 64 m + 60 < nblocks
        const int j = w & 3, whole = nblocks > j + 60 ? (nblocks - j - 61) / 64 + 1 : 0;
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = src[(long long)(k < 4 * whole ? w + 16 * k : 0) * kPartStride];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc += k < 4 * whole ? v[k] : 0.f;
        const int b0 = j + 64 * whole;
        if (w < 4 && b0 < nblocks) {
#pragma unroll
            for (int k = 0; k < 15; ++k) v[k] = src[(long long)(b0 + 4 * k < nblocks ? b0 + 4 * k : 0) * kPartStride];
#pragma unroll
            for (int k = 0; k < 15; ++k) acc += b0 + 4 * k < nblocks ? v[k] : 0.f;
        }
    }
    red[w][lane] = acc;
    __syncthreads();
    if (w != 0 || p > kNParam) return;
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = (red[j][lane] + red[j + 4][lane]) + (red[j + 8][lane] + red[j + 12][lane]);
    const float gr = (t[0] + t[1]) + (t[2] + t[3]);
    grad[p] = gr;
    if (mine) {
        const float a = fmaf(1.f - A.beta1, gr, A.beta1 * m1);
        const float b = fmaf(gr, (1.f - A.beta2) * gr, A.beta2 * m2);
        A.m1[p] = a;
        A.m2[p] = b;
        A.P[p] = P0 - A.lr * (a / A.bc1) / (sqrtf(b / A.bc2) + A.eps);
    }
}

// --------------------------------------------------- closure in the fluid --
// Judge: sums over cells of |q_net - q_kin|^2 and |q_kin|^2 (q_i = Q_ijj),
// per block in a fixed order.
__global__ void __launch_bounds__(256)
mlp_judge_partial_kernel(MlpSet S, const double* __restrict__ scale, const float* __restrict__ y, long long cells,
                         double* __restrict__ part) {
    const int sp = blockIdx.y;
    const double* __restrict__ M = S.M[sp];
    const double m = S.m[sp];
    scale += (size_t)sp * cells;
    y += (size_t)sp * cells * kOutPad;
    part += (size_t)sp * 2 * gridDim.x;
    __shared__ double red[2 * 4];
    double e2 = 0.0, k2 = 0.0;
    for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < cells;
         c += (long long)gridDim.x * blockDim.x) {
        double Q[10], n, u[3], Tref;
        heat_flux_cell(M, c, m, Q, n, u, Tref);
        const double qk[3] = {Q[0] + Q[3] + Q[5], Q[1] + Q[6] + Q[8], Q[2] + Q[7] + Q[9]};
        const double sc = scale[c];
        const float* yc = y + c * 16;
        const double qn[3] = {sc * ((double)yc[0] + (double)yc[3] + (double)yc[5]),
                              sc * ((double)yc[1] + (double)yc[6] + (double)yc[8]),
                              sc * ((double)yc[2] + (double)yc[7] + (double)yc[9])};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            e2 += (qn[d] - qk[d]) * (qn[d] - qk[d]);
            k2 += qk[d] * qk[d];
        }
    }
    double v[2] = {e2, k2};
    block_sum<2>(v, red);
    if (threadIdx.x == 0) {
        part[blockIdx.x * 2] = v[0];
        part[blockIdx.x * 2 + 1] = v[1];
    }
}

// One wave per species: lane l adds partials l, l + 64, ... (the loads of
// all lanes in flight together), then a butterfly over the wave: a fixed
// order of additions on every call.
__global__ void __launch_bounds__(64)
mlp_judge_finish_kernel(MlpSet S, const double* __restrict__ part, int nblocks, double tol) {
    const int sp = blockIdx.x, lane = threadIdx.x;
    int* __restrict__ fallback = S.fallback[sp];
    double* __restrict__ err = S.err[sp];
    part += (size_t)sp * 2 * nblocks;
    double e2 = 0.0, k2 = 0.0;
    for (int b = lane; b < nblocks; b += 64) {
        e2 += part[2 * b];
        k2 += part[2 * b + 1];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        e2 += __shfl_xor(e2, o, 64);
        k2 += __shfl_xor(k2, o, 64);
    }
    if (lane != 0) return;
    const double r = sqrt(e2) / fmax(sqrt(k2), 1e-300);
    *err = r;
    *fallback = !(r <= tol);
}

// --------------------------------------------------------------- launchers --
constexpr int kJudgeBlocks = 256;

hipError_t launch_mlp_features_set(const MlpSet& S, int ns, int s0, int stride, const double* B, int nx, int ny,
                                   unsigned short* x, double* scale, hipStream_t st) {
    if (ns < 1 || ns > 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mlp_features_kernel<false>, dim3((nx + kFeatCols - 1) / kFeatCols, (ny + kFeatRows - 1) / kFeatRows, ns),
                       dim3(2 * kFeatCells), 0, st, S, s0, stride, B, nx, ny, x, scale, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_mlp_network_set(const MlpSet& S, int ns, int s0, int stride, const double* B, int nx, int ny,
                                  const float* params, double* scale, float* y, hipStream_t st) {
    if (ns < 1 || ns > 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mlp_features_kernel<true>, dim3((nx + kFeatCols - 1) / kFeatCols, (ny + kFeatRows - 1) / kFeatRows, ns),
                       dim3(2 * kFeatCells), 0, st, S, s0, stride, B, nx, ny, nullptr, scale, params, y);
    return hipGetLastError();
}

hipError_t launch_mlp_features(const double* M, int stride, const double* B, int nx, int ny, double m, int species,
                               unsigned short* x, double* scale, hipStream_t st) {
    MlpSet S{};
    S.M[0] = M;
    S.m[0] = m;
    return launch_mlp_features_set(S, 1, species, stride, B, nx, ny, x, scale, st);
}

hipError_t launch_mlp_targets(const double* M, long long cells, double m, float* y, hipStream_t st) {
    hipLaunchKernelGGL(mlp_targets_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, st, M, cells, m, y);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float* P, const unsigned short* x, long long n, float* y, hipStream_t st) {
    const long long tiles = (n + 15) / 16;
    long long blocks = (tiles + 3) / 4;
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(mlp_forward_kernel, dim3((unsigned)blocks), dim3(256), 0, st, P, x, n, y);
    return hipGetLastError();
}

// At most one gradient block per compute unit: every block stages the whole
// network in LDS first, so fewer blocks with more tiles each beat more blocks
// (16384-row batches, gradient + sum + Adam: 256 blocks 1.4x faster than 512
// and 1.25x faster than 128).
constexpr long long kGradBlocks = 256;      // mlp_reduce_kernel adds at most this many
size_t mlp_grad_blocks(long long n) {
    const long long tiles = (n + 15) / 16;
    long long blocks = tiles < kGradBlocks ? tiles : kGradBlocks;
    return blocks < 1 ? 1 : (size_t)blocks;
}
size_t mlp_part_floats(long long n) { return mlp_grad_blocks(n) * (size_t)kPartStride; }

static AdamArgs adam_args(float* P, float* m1, float* m2, long long step, double lr) {
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    const double bc1 = 1.0 - pow(b1, (double)step), bc2 = 1.0 - pow(b2, (double)step);
    return AdamArgs{P, m1, m2, (float)lr, (float)b1, (float)b2, (float)eps, (float)bc1, (float)bc2};
}

static hipError_t grad_and_sum(const float* P, const unsigned short* x, const float* t, long long n, float* part,
                               float* grad, hipStream_t st, const long long* idx, long long nrows,
                               const AdamArgs& A) {
    const long long tiles = (n + 15) / 16;
    const long long blocks = (long long)mlp_grad_blocks(n);
    const long long tpb = (tiles + blocks - 1) / blocks;
    const float inv_norm = (float)(1.0 / ((double)n * kOut));
    hipLaunchKernelGGL(mlp_grad_kernel, dim3((unsigned)blocks), dim3(512), 0, st, P, x, t, n, tpb, inv_norm, part,
                       idx, nrows);
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3((kNParam + 1 + 63) / 64), dim3(1024), 0, st, part, (int)blocks, grad,
                       A);
    return hipGetLastError();
}

hipError_t launch_mlp_gradient(const float* P, const unsigned short* x, const float* t, long long n, float* part,
                               float* grad, hipStream_t st, const long long* idx, long long nrows) {
    return grad_and_sum(P, x, t, n, part, grad, st, idx, nrows, AdamArgs{});
}

hipError_t launch_mlp_train_step(float* P, float* m1, float* m2, long long step, double lr,
                                 const unsigned short* x, const float* t, long long n, float* part, float* grad,
                                 hipStream_t st, const long long* idx, long long nrows) {
    return grad_and_sum(P, x, t, n, part, grad, st, idx, nrows, adam_args(P, m1, m2, step, lr));
}

size_t mlp_judge_part_doubles() { return 2 * kJudgeBlocks; }

hipError_t launch_mlp_judge_set(const MlpSet& S, int ns, const double* scale, const float* y, long long cells,
                                double tol, double* part, hipStream_t st) {
    if (ns < 1 || ns > 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(mlp_judge_partial_kernel, dim3(kJudgeBlocks, ns), dim3(256), 0, st, S, scale, y, cells, part);
    hipLaunchKernelGGL(mlp_judge_finish_kernel, dim3(ns), dim3(64), 0, st, S, part, kJudgeBlocks, tol);
    return hipGetLastError();
}

}  // namespace vl
