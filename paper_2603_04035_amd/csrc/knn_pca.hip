// PCA of the rows of X to p dimensions, the preprocessing the paper applies
// before its k-NN stage (pca_dim; sections "Reproducibility" and "Scaling
// Behavior"), in FP64 from the stored values:
//
//  1. mean:     column sums over fixed row chunks, then summed in chunk order;
//  2. Gram:     C = (X - mu)^T (X - mu) / (n - 1) on v_mfma_f64_16x16x4_f64,
//               upper-triangle 64x64 tiles, one partial per 4096-row chunk
//               (rows staged in LDS as FP32, centred as they become
//               operands), partials summed in chunk order: no atomics, so
//               the result does not depend on scheduling;
//  3. subspace: m = min(d, 80, max(2p, p + 16)) columns V (seeded, hashed
//               values) are filtered by Chebyshev polynomials of C that damp
//               the eigenvalues below the block's smallest Rayleigh quotient
//               (Zhou and Saad 2007): rounds of q products C Y on
//               v_mfma_f64_16x16x4_f64, each round ended by one shifted
//               Cholesky-QR pass on columns scaled to norm 1, and after the
//               last by shifted + two plain passes (Cholesky-QR3); then
//               Rayleigh-Ritz: H = V^T C V, whose eigenpairs come from cyclic
//               Jacobi rotations (one workgroup, round-robin pairing), and
//               the p largest Ritz pairs are kept; each eigenvector's entry
//               of largest magnitude is made positive;
//  4. project:  Z = (X - mu) V_p, rounded to FP32.
// When m = d the Ritz pairs are the exact eigenpairs of C.
#include <math.h>

#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "knn_common.hpp"

namespace knn {

constexpr int kPcaMaxP = 64;      // components
constexpr int kPcaMaxM = 80;      // subspace width (an m x m double matrix fits in LDS)
static_assert(kPcaMaxM % 16 == 0, "LDS kernels stride columns by 16");
constexpr int kPcaChunk = 4096;   // rows per Gram partial
constexpr int kPcaSumChunk = 512; // rows per column-sum partial
constexpr int kPcaMaxQ = 8;       // products C V between orthonormalisations, at most
constexpr int kPcaTile = 64;      // Gram tile edge

typedef double f64x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ mean

// part[c][t] = sum of column t over rows [c * kPcaSumChunk, ...), in row order
// (thread t of a 256-wide column block walks the chunk's rows).
template <int DT>
__global__ __launch_bounds__(256) void pca_colsum_kernel(const void* __restrict__ X, int64_t n, int64_t ld, int d,
                                                         double* __restrict__ part)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    const int64_t c = blockIdx.y;
    if (t >= d) return;
    const int64_t r0 = c * kPcaSumChunk, r1 = r0 + kPcaSumChunk < n ? r0 + kPcaSumChunk : n;
    double s = 0.0;
    for (int64_t r = r0; r < r1; ++r) s += (double)elem<DT>::ld(X, r * ld + t);
    part[c * d + t] = s;
}

__global__ __launch_bounds__(256) void pca_mean_kernel(const double* __restrict__ part, int nch, int d, int64_t n,
                                                       double* __restrict__ mu)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= d) return;
    double s = 0.0;
    for (int c = 0; c < nch; ++c) s += part[(int64_t)c * d + t];
    mu[t] = s / (double)n;
}

// ------------------------------------------------------------------ Gram

// Tile (ta, tb), ta <= tb, of chunk c: G[a][b] over the chunk's rows for
// columns a in [64 ta, +64), b in [64 tb, +64).  Rows are staged 64 at a
// time (FP32, both column slices).  Wave w owns tile rows 16w .. 16w+15 and
// all 64 tile columns: four 16x16 f64 accumulators.  v_mfma_f64_16x16x4:
// lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator item
// i of lane l is D[l / 16 + 4 i][l % 16] (rows interleaved by 4).
template <int DT>
__global__ __launch_bounds__(256) void pca_gram_kernel(const void* __restrict__ X, int64_t n, int64_t ld, int d,
                                                       const double* __restrict__ mu, const int2* __restrict__ tiles,
                                                       double* __restrict__ part)
{
    __shared__ float sa[64][kPcaTile + 1];
    __shared__ float sb[64][kPcaTile + 1];
    __shared__ double sma[kPcaTile], smb[kPcaTile];
    const int2 tt = tiles[blockIdx.x];
    const int64_t c = blockIdx.y;
    const int a0 = tt.x * kPcaTile, b0 = tt.y * kPcaTile;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t r0 = c * kPcaChunk, r1 = r0 + kPcaChunk < n ? r0 + kPcaChunk : n;
    if (tid < kPcaTile) {
        sma[tid] = a0 + tid < d ? mu[a0 + tid] : 0.0;
        smb[tid] = b0 + tid < d ? mu[b0 + tid] : 0.0;
    }
    // staging: thread (rq, cc) holds rows rq, rq + 4, ..., rq + 60 of column
    // cc of both slices; the next 64 rows are loaded while this step's
    // MFMAs run (zeros past d and past the chunk)
    const int cc = tid & 63, rq = tid >> 6;
    const bool acol = a0 + cc < d, bcol = b0 + cc < d;
    float pa[16], pb[16];
    auto fetch = [&](int64_t rs) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int64_t row = rs + rq + 4 * u;
            const bool ok = row < r1;
            pa[u] = ok && acol ? elem<DT>::ld(X, row * ld + a0 + cc) : 0.0f;
            pb[u] = ok && bcol ? elem<DT>::ld(X, row * ld + b0 + cc) : 0.0f;
        }
    };
    fetch(r0);
    f64x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int ia = 16 * w + (lane & 15);
    for (int64_t rs = r0; rs < r1; rs += 64) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            sa[rq + 4 * u][cc] = pa[u];
            sb[rq + 4 * u][cc] = pb[u];
        }
        __syncthreads();
        if (rs + 64 < r1) fetch(rs + 64);
        const int nr = (int)(r1 - rs < 64 ? r1 - rs : 64);
#pragma unroll 4
        for (int k0 = 0; k0 < 64; k0 += 4) {
            const int kk = k0 + (lane >> 4);
            const bool kv = kk < nr;
            // centred operands; padded rows and columns contribute 0
            const float xa = sa[kk][ia];
            const double av = kv ? (double)xa - sma[ia] : 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int jb = 16 * j + (lane & 15);
                const float xb = sb[kk][jb];
                const double bv = kv ? (double)xb - smb[jb] : 0.0;
                acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[j], 0, 0, 0);
            }
        }
    }
    // partial tile, full 64 x 64 block of the chunk's d x d matrix
    double* out = part + c * (int64_t)d * d;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ra = a0 + 16 * w + (lane >> 4) + 4 * i, cb = b0 + 16 * j + (lane & 15);
            if (ra < d && cb < d) out[(int64_t)ra * d + cb] = acc[j][i];
        }
    }
}

// C[a][b] = sum of the chunk partials (chunk order) / (n - 1) for a <= b
// (inside the upper tiles computed), mirrored to C[b][a].
__global__ __launch_bounds__(256) void pca_gram_reduce_kernel(const double* __restrict__ part, int nch, int d,
                                                              int64_t n, double* __restrict__ C)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)d * d) return;
    const int a = (int)(e / d), b = (int)(e % d);
    if (a > b) return;   // the lower triangle is mirrored from the upper one
    double s = 0.0;
    for (int c = 0; c < nch; ++c) s += part[(int64_t)c * d * d + e];
    s /= (double)(n - 1);
    C[(int64_t)a * d + b] = s;
    C[(int64_t)b * d + a] = s;
}

// ------------------------------------------------------------------ subspace

// V (m columns of length d, column-major) from hashed values in [-1, 1).
__global__ __launch_bounds__(256) void pca_init_kernel(int d, int m, uint64_t seed, double* __restrict__ V)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)d * m) return;
    V[e] = 2.0 * ((double)(hash4(seed, 11, (uint64_t)e, 0) >> 11) * (1.0 / 9007199254740992.0)) - 1.0;
}

// V = the first m columns of the d x d identity (column-major).
__global__ __launch_bounds__(256) void pca_identity_kernel(int d, int m, double* __restrict__ V)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)d * m) return;
    V[e] = (e / d == e % d) ? 1.0 : 0.0;
}

// W = alpha (C V - shift V) - P on v_mfma_f64_16x16x4_f64 (P nullable; alpha
// = 1, shift = 0: the plain product), one workgroup per 16 x 16 block of W
// (rows a of C, columns j of V).  K runs in blocks of 16, block b taken by
// wave b % 4 (four blocks per round, loads first): lane l (r = l % 16, g = l / 16) holds C[a0 + r][k0 + 4g ..
// +3] and V[j0 + r][k0 + 4g .. +3], and step s multiplies the k = k0 + 4g +
// s slice, so every k enters once; entries past d or m are zero.  The four
// waves' sums are added in wave order.  Accumulator item i of lane l is
// W[j0 + r][a0 + g + 4i].
__global__ __launch_bounds__(256) void pca_cv_kernel(const double* __restrict__ C, const double* __restrict__ V, int d,
                                                     int m, double alpha, double shift, const double* P, double* W)
{
    __shared__ double part[3][64][4];
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, r = l & 15, g = l >> 4;
    const int a0 = blockIdx.x * 16, j0 = blockIdx.y * 16;
    const bool aok = a0 + r < d, jok = j0 + r < m;
    const double* crow = C + (int64_t)(aok ? a0 + r : 0) * d;
    const double* vcol = V + (int64_t)(jok ? j0 + r : 0) * d;
    f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
    // four of the wave's K blocks per round, all their loads issued first
    for (int kb = 16 * wv; kb < d; kb += 256) {
        double ca[4][4], vb[4][4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = kb + 64 * b + 4 * g + s;
                ca[b][s] = aok && k < d ? crow[k] : 0.0;
                vb[b][s] = jok && k < d ? vcol[k] : 0.0;
            }
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[b][s], vb[b][s], acc, 0, 0, 0);
    }
    if (wv > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) part[wv - 1][l][i] = acc[i];
    }
    __syncthreads();
    if (wv == 0 && jok) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double v = ((acc[i] + part[0][l][i]) + part[1][l][i]) + part[2][l][i];
            const int a = a0 + g + 4 * i;
            if (a < d) {
                const int64_t e = (int64_t)(j0 + r) * d + a;   // P may be W itself
                double x = shift != 0.0 ? v - shift * V[e] : v;
                x = alpha != 1.0 ? alpha * x : x;
                W[e] = P ? x - P[e] : x;
            }
        }
    }
}

// S[i][j] = <W_i, W_j> over d (i <= j; mirrored), one workgroup per pair,
// a fixed-order tree over the 256 thread sums.
__global__ __launch_bounds__(256) void pca_gram_small_kernel(const double* __restrict__ W, const double* __restrict__ U,
                                                             int d, int m, double* __restrict__ S)
{
    __shared__ double red[256];
    const int i = blockIdx.x, j = blockIdx.y;
    if (U == W && i > j) return;
    const double* wi = U + (int64_t)i * d;
    const double* wj = W + (int64_t)j * d;
    double s = 0.0;
    for (int a = threadIdx.x; a < d; a += 256) s = fma(wi[a], wj[a], s);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        S[i * m + j] = red[0];
        if (U == W) S[j * m + i] = red[0];
    }
}

// out[j] = <V_j, Y_j>, out[m + j] = <V_j, V_j> (one workgroup per column, a
// fixed-order tree): the columns' Rayleigh quotients when Y = C V.
__global__ __launch_bounds__(256) void pca_rayleigh_kernel(const double* __restrict__ V, const double* __restrict__ Y,
                                                           int d, int m, double* __restrict__ out)
{
    __shared__ double ra[256], rb[256];
    const int j = blockIdx.x, t = threadIdx.x;
    double a = 0.0, b = 0.0;
    for (int i = t; i < d; i += 256) {
        const double v = V[(int64_t)j * d + i];
        a = fma(v, Y[(int64_t)j * d + i], a);
        b = fma(v, v, b);
    }
    ra[t] = a;
    rb[t] = b;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) {
            ra[t] += ra[t + o];
            rb[t] += rb[t + o];
        }
        __syncthreads();
    }
    if (t == 0) {
        out[j] = ra[0];
        out[m + j] = rb[0];
    }
}

// out[k] = C[k][k] (a strided copy to the host takes 5 ms for 784 of them).
__global__ __launch_bounds__(256) void pca_diag_kernel(const double* __restrict__ C, int d, double* __restrict__ out)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < d) out[k] = C[(int64_t)k * d + k];
}

// One Cholesky-QR pass: V = W R^{-1}, where S = W^T W = R^T R (R upper
// triangular).  Every workgroup factors S (its entries in registers, 25 per
// thread), the same operations in each, so all hold the same factor; then
// it forms 64 rows of W R^{-1} for its eight columns.  The factor comes from
// symmetric elimination on [S | I] (one barrier per step, the pivot row
// passed through LDS): step k subtracts
// S[k][i] / S[k][k] times row k from each row i > k, on the trailing upper
// triangle of S and on the unit lower triangular M beside it, so that at
// the end M S = D L^T with S = L D L^T (L unit lower triangular, D the
// pivots) and M = L^{-1}.  Then R = D^{1/2} L^T and R^{-1}[i][j] = M[j][i] /
// sqrt(D[j]): no triangular solve is needed.  M's strict lower triangle sits
// in the lower half of S, which the upper-triangle elimination never reads.
// The columns of W are first scaled to norm 1 (S to unit diagonal; a zero
// column stays): filtered columns differ by many orders of magnitude in length
// alone, which then costs nothing.  With shift_rel > 0 the factored matrix is
// S + s I, s = shift_rel * m (shifted Cholesky-QR: V spans the same
// space as W, but is only near-orthonormal, and no pivot can fail however
// badly W is conditioned).  A non-positive pivot (W of lower rank than m,
// unshifted) is replaced by 1 and flagged, which keeps the factor finite.
// The pivots D[k] (as used) go to `pivots`: their spread estimates W's
// conditioning.
constexpr int kPcaCols = 8;

__global__ __launch_bounds__(256) void pca_cholqr_kernel(const double* __restrict__ Sg, const double* __restrict__ W,
                                                         int d, int m, double* __restrict__ V,
                                                         unsigned* __restrict__ bad, double* __restrict__ pivots,
                                                         double shift_rel)
{
    __shared__ double S[kPcaMaxM * kPcaMaxM];   // the result: upper R-scaled rows, strict lower M
    __shared__ double rowk[2][kPcaMaxM];         // the step's pivot row (double-buffered)
    __shared__ double rinv[kPcaMaxM];
    __shared__ double dinv[kPcaMaxM];            // the columns' scales
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    // thread (ty, tx) owns entries (ty + 16u, tx + 16q), u, q < NJ, held in
    // registers through the whole elimination; only the pivot row of each
    // step goes through LDS (one barrier per step)
    constexpr int NJ = kPcaMaxM / 16;
    if (tid < m) {
        const double v = Sg[tid * m + tid];
        dinv[tid] = v > 0.0 ? 1.0 / sqrt(v) : 1.0;
    }
    __syncthreads();
    double x[NJ][NJ];
#pragma unroll
    for (int u = 0; u < NJ; ++u)
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            const int i = ty + 16 * u, j = tx + 16 * q;
            x[u][q] = i < m && j < m && j >= i ? Sg[i * m + j] * dinv[i] * dinv[j] : 0.0;
            // S + s I: the same span, positive pivots however badly W is conditioned
            if (i == j && i < m) x[u][q] += shift_rel * (double)m;
        }
    if (ty == 0) {
#pragma unroll
        for (int q = 0; q < NJ; ++q) rowk[0][tx + 16 * q] = x[0][q];
    }
    // 16 steps at a time, so that what a step does to each 16 x 16 block of
    // entries is known: rows below the steps' block take row k's entry in the
    // columns before it and from the diagonal on, nothing in between; only
    // blocks on the steps' row or column or on the diagonal ask per entry
    // (80 columns: 81 us a pass with every entry asking, 52 so).
#pragma unroll
    for (int kb = 0; kb < NJ; ++kb) {
        for (int kk = 0; kk < 16; ++kk) {
            const int k = 16 * kb + kk;
            if (k >= m) break;
            __syncthreads();
            const double* rk = rowk[k & 1];
            double pk = rk[k];
            if (!(pk > 0.0)) {
                if (tid == 0 && blockIdx.x == 0 && blockIdx.y == 0) atomicOr(bad, 1u);
                pk = 1.0;
            }
            const double ip = 1.0 / pk;
            double rkq[NJ], fu[NJ];
#pragma unroll
            for (int q = 0; q < NJ; ++q) rkq[q] = rk[tx + 16 * q];
#pragma unroll
            for (int u = kb; u < NJ; ++u) fu[u] = rk[ty + 16 * u] * ip;
#pragma unroll
            for (int u = kb; u < NJ; ++u)
#pragma unroll
                for (int q = 0; q < NJ; ++q) {
                    if (u > kb && q > kb && q < u) continue;   // k < j < i
                    if (u > kb && (q < kb || q > u)) {
                        x[u][q] = fma(-fu[u], rkq[q], x[u][q]);
                        continue;
                    }
                    const int i = ty + 16 * u, j = tx + 16 * q;
                    // rows below k: the upper triangle (j >= i) and M (j < k) take
                    // row k's entry; M's column k takes its unit diagonal; k < j < i
                    // stays 0
                    const double nv = (j >= i || j < k) ? fma(-fu[u], rkq[q], x[u][q])
                                                        : (j == k ? x[u][q] - fu[u] : x[u][q]);
                    x[u][q] = i > k ? nv : x[u][q];
                }
            if (tid == 0) {
                rinv[k] = 1.0 / sqrt(pk);
                if (blockIdx.x == 0 && blockIdx.y == 0) pivots[k] = pk;
            }
            // row k + 1 is final now: its owners publish it for the next step
            const int k1 = k + 1;
            if (k1 < m && ty == (k1 & 15)) {
                if (kk < 15) {
#pragma unroll
                    for (int q = 0; q < NJ; ++q) rowk[k1 & 1][tx + 16 * q] = x[kb][q];
                } else if (kb + 1 < NJ) {
#pragma unroll
                    for (int q = 0; q < NJ; ++q) rowk[k1 & 1][tx + 16 * q] = x[kb + 1 < NJ ? kb + 1 : kb][q];
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NJ; ++u)
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            const int i = ty + 16 * u, j = tx + 16 * q;
            // M's column j multiplies column j of W: its scale goes in here
            if (i < m && j < m) S[i * m + j] = i > j ? x[u][q] * dinv[j] : (i == j ? dinv[i] : x[u][q]);
        }
    __syncthreads();
    // V = W R^{-1} for rows a0 .. a0 + 63 and the workgroup's eight columns:
    // wave g sums the products over its quarter of the index range i (so
    // each thread issues a quarter of the row loads), and the four partial
    // sums are added in wave order
    const int r = tid & 63, g = tid >> 6;
    const int a = blockIdx.x * 64 + r;
    const int j0 = blockIdx.y * kPcaCols;
    const int jmax = j0 + kPcaCols < m ? j0 + kPcaCols : m;
    const int ilen = (jmax + 3) / 4, ib = g * ilen, ie = ib + ilen < jmax ? ib + ilen : jmax;
    double sp[kPcaCols];
#pragma unroll
    for (int q = 0; q < kPcaCols; ++q) sp[q] = 0.0;
    if (a < d) {
        for (int i0 = ib; i0 < ie; i0 += 8) {
            double wv[8];   // eight rows of W in flight at once
#pragma unroll
            for (int u = 0; u < 8; ++u) wv[u] = i0 + u < ie ? W[(int64_t)(i0 + u) * d + a] : 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u;
#pragma unroll
                for (int q = 0; q < kPcaCols; ++q) {
                    const int j = j0 + q;
                    if (i < ie && j < m && i <= j) sp[q] = fma(wv[u], S[j * m + i], sp[q]);
                }
            }
        }
    }
    __shared__ double part[3][64][kPcaCols];
    if (g > 0) {
#pragma unroll
        for (int q = 0; q < kPcaCols; ++q) part[g - 1][r][q] = sp[q];
    }
    __syncthreads();
    if (g == 0 && a < d) {
#pragma unroll
        for (int q = 0; q < kPcaCols; ++q)
            if (j0 + q < m)
                V[(int64_t)(j0 + q) * d + a] = (((sp[q] + part[0][r][q]) + part[1][r][q]) + part[2][r][q]) * rinv[j0 + q];
    }
}

// Cyclic Jacobi on the symmetric m x m matrix H (row-major; H and the
// transposed rotations E^T held in LDS, copied back at the end), one
// workgroup: each sweep runs m - 1 rounds of the round-robin tournament
// (m even; an odd m plays a bye), every round rotating its m/2 disjoint
// pairs (p, q) so that H[p][q] becomes 0, with E accumulating the rotations (E
// starts as the identity).  Thread (s, t), s <= t, rotates the 2 x 2 block of
// rows p_s, q_s and columns p_t, q_t from both sides at once and writes it
// with its mirror image: the blocks are disjoint, so a round needs one pass
// and two barriers.  A round is latency (the angles' square roots and
// divisions, the barriers): with rows and columns in separate passes by 256
// threads the eigenproblem of an 80-wide block took 2.09 ms, 1.04 now.  Sweeps
// stop when the sum of H[i][j]^2 / (H[i][i] H[j][j]) off the diagonal falls
// below 1e-26 (entries below 1e-13 of the eigenvalues they would mix: against
// the whole norm, a leading eigenvalue 10^6 times the rest left the rest's
// vectors off by 10^-7), when the off-diagonal mass is below 1e-33 of the total
// (rounding), or after 40.
constexpr int kJacThreads = 1024;

__global__ __launch_bounds__(kJacThreads) void pca_jacobi_kernel(double* __restrict__ Hg, double* __restrict__ Eg, int m)
{
    __shared__ double H[kPcaMaxM * kPcaMaxM];
    __shared__ double E[kPcaMaxM * kPcaMaxM];   // E^T: row j is column j of E
    __shared__ double cs[kPcaMaxM / 2], sn[kPcaMaxM / 2];
    __shared__ int pp[kPcaMaxM / 2], qq[kPcaMaxM / 2];
    __shared__ double red[3][kJacThreads / 64];
    const int tid = threadIdx.x;
    // V^T (C V) is symmetric up to rounding: take its symmetric part
    for (int e = tid; e < m * m; e += kJacThreads) {
        H[e] = 0.5 * (Hg[e] + Hg[(e % m) * m + e / m]);
        E[e] = (e / m == e % m) ? 1.0 : 0.0;
    }
    const int mm = m + (m & 1), np = mm / 2;   // players, with a bye for odd m
    // this thread's block (s, t), s <= t < np, of the np (np + 1) / 2 <= 820
    int bs = -1, bt = 0;
    {
        int e = tid;
        for (int t = 0; t < np && bs < 0; ++t) {
            if (e <= t) {
                bs = e;
                bt = t;
            }
            e -= t + 1;
        }
    }
    for (int sweep = 0; sweep < 40; ++sweep) {
        __syncthreads();
        double off = 0.0, tot = 0.0, rel = 0.0;
        for (int e = tid; e < m * m; e += kJacThreads) {
            const double h = H[e], h2 = h * h;
            const int i = e / m, j = e - i * m;
            tot += h2;
            if (i != j && h2 > 0.0) {
                off += h2;
                rel += h2 / fabs(H[i * m + i] * H[j * m + j]);
            }
        }
        for (int o = 32; o > 0; o >>= 1) {
            off += __longlong_as_double((long long)shfl_xor_u64((uint64_t)__double_as_longlong(off), o));
            tot += __longlong_as_double((long long)shfl_xor_u64((uint64_t)__double_as_longlong(tot), o));
            rel += __longlong_as_double((long long)shfl_xor_u64((uint64_t)__double_as_longlong(rel), o));
        }
        if ((tid & 63) == 0) {
            red[0][tid >> 6] = off;
            red[1][tid >> 6] = tot;
            red[2][tid >> 6] = rel;
        }
        __syncthreads();
        off = tot = rel = 0.0;
        for (int w = 0; w < kJacThreads / 64; ++w) {
            off += red[0][w];
            tot += red[1][w];
            rel += red[2][w];
        }
        if (!(off > 1e-33 * tot) || rel <= 1e-26) break;
        for (int round = 0; round < mm - 1; ++round) {
            // pairs of this round: player 0 fixed, the others rotate
            if (tid < np) {
                int a = tid == 0 ? 0 : 1 + (round + tid - 1) % (mm - 1);
                int b = 1 + (round + mm - 2 - tid) % (mm - 1);
                if (a > b) {
                    const int x = a;
                    a = b;
                    b = x;
                }
                pp[tid] = a;
                qq[tid] = b;
                double c = 1.0, s = 0.0;
                if (b < m) {
                    const double apq = H[a * m + b];
                    if (apq != 0.0) {
                        const double theta = (H[b * m + b] - H[a * m + a]) / (2.0 * apq);
                        const double tt = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
                        c = 1.0 / sqrt(tt * tt + 1.0);
                        s = tt * c;
                    }
                }
                cs[tid] = c;
                sn[tid] = s;
            }
            __syncthreads();
            if (bs >= 0) {
                const int p1 = pp[bs], q1 = qq[bs], p2 = pp[bt], q2 = qq[bt];
                const bool o1 = q1 < m, o2 = q2 < m;   // not the bye
                const double c1 = cs[bs], s1 = sn[bs], c2 = cs[bt], s2 = sn[bt];
                const double x00 = H[p1 * m + p2], x01 = o2 ? H[p1 * m + q2] : 0.0;
                const double x10 = o1 ? H[q1 * m + p2] : 0.0, x11 = o1 && o2 ? H[q1 * m + q2] : 0.0;
                const double r00 = c1 * x00 - s1 * x10, r01 = c1 * x01 - s1 * x11;
                const double r10 = s1 * x00 + c1 * x10, r11 = s1 * x01 + c1 * x11;
                const double y00 = c2 * r00 - s2 * r01, y01 = s2 * r00 + c2 * r01;
                const double y10 = c2 * r10 - s2 * r11, y11 = s2 * r10 + c2 * r11;
                H[p1 * m + p2] = y00;
                H[p2 * m + p1] = y00;
                if (o2) {
                    H[p1 * m + q2] = y01;
                    H[q2 * m + p1] = y01;
                }
                if (o1 && (bs != bt)) {
                    H[q1 * m + p2] = y10;
                    H[p2 * m + q1] = y10;
                }
                if (o1 && o2) {
                    H[q1 * m + q2] = y11;
                    H[q2 * m + q1] = y11;
                }
            }
            for (int e = tid; e < np * m; e += kJacThreads) {
                const int t = e / m, i = e - t * m, p = pp[t], q = qq[t];
                if (q < m) {
                    const double c = cs[t], s = sn[t], ep = E[p * m + i], eq = E[q * m + i];
                    E[p * m + i] = c * ep - s * eq;
                    E[q * m + i] = s * ep + c * eq;
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();
    for (int e = tid; e < m * m; e += kJacThreads) {
        Hg[e] = H[e];
        Eg[(e % m) * m + e / m] = E[e];
    }
}

// The p largest Ritz pairs: eigenvalues from diag(H) sorted descending
// (ties by index), vectors U_j = V e_j (e_j a column of E), each sign-fixed
// so that its entry of largest magnitude (the first such) is positive.
// Workgroup j forms component j; U is d x p row-major, lam has p entries.
// With `bad` (the subspace is not all of R^d) a smallest Ritz value below
// 1e-12 of the largest flags an X of lower rank than m (its noise level is
// some 1e-16 of the largest for exact inputs, 1e-14 for rounded ones).
__global__ __launch_bounds__(256) void pca_ritz_kernel(const double* __restrict__ H, const double* __restrict__ E,
                                                       const double* __restrict__ V, int d, int m, int p,
                                                       double* __restrict__ U, double* __restrict__ lam,
                                                       unsigned* __restrict__ bad)
{
    __shared__ double ecol[kPcaMaxM];
    __shared__ double red[256];
    __shared__ int redi[256];
    __shared__ int col_;
    const int tid = threadIdx.x, j = blockIdx.x;
    if (tid < m) {
        const double x = H[tid * m + tid];
        int rank = 0;
        double top = x;
        for (int q = 0; q < m; ++q) {
            const double y = H[q * m + q];
            rank += (y > x || (y == x && q < tid)) ? 1 : 0;
            top = y > top ? y : top;
        }
        if (rank == j) col_ = tid;
        if (bad && j == 0 && !(x > 1e-12 * top)) atomicOr(bad, 2u);
    }
    __syncthreads();
    const int col = col_;
    if (tid < m) ecol[tid] = E[tid * m + col];
    __syncthreads();
    double best = -1.0;
    int bi = 0;
    for (int a = tid; a < d; a += 256) {
        double s = 0.0;
        for (int i = 0; i < m; ++i) s = fma(V[(int64_t)i * d + a], ecol[i], s);
        if (fabs(s) > best) {
            best = fabs(s);
            bi = a;
        }
        U[(int64_t)a * p + j] = s;
    }
    red[tid] = best;
    redi[tid] = bi;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o && (red[tid + o] > red[tid] || (red[tid + o] == red[tid] && redi[tid + o] < redi[tid]))) {
            red[tid] = red[tid + o];
            redi[tid] = redi[tid + o];
        }
        __syncthreads();
    }
    const double sg = U[(int64_t)redi[0] * p + j] < 0.0 ? -1.0 : 1.0;
    if (tid == 0) lam[j] = H[col * m + col];
    for (int a = tid; a < d; a += 256) U[(int64_t)a * p + j] *= sg;
}

// Z[r][j] = sum_t (x_rt - mu_t) U[t][j] on v_mfma_f64_16x16x4_f64, rounded
// to FP32: wave w of workgroup b takes rows 16 (4b + w) .. +15 and every
// 16-column block of U (p <= 64: up to four accumulators), so each row of X
// is read once.  K runs as in pca_cv_kernel (lane l holds coordinates
// k0 + 4 (l / 16) .. +3 of row l % 16, step s takes the k0 + 4g + s slice).
template <int DT>
__global__ __launch_bounds__(256) void pca_project_kernel(const void* __restrict__ X, int64_t n, int64_t ld, int d,
                                                          const double* __restrict__ mu, const double* __restrict__ U,
                                                          int p, float* __restrict__ Z)
{
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, r = l & 15, g = l >> 4;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + wv) * 16;
    if (row0 >= n) return;   // the whole wave
    const int64_t row = row0 + r;
    const bool rok = row < n;
    const int nt = (p + 15) / 16;
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    // two K blocks per round, the row's loads issued first
    for (int kb = 0; kb < d; kb += 32) {
        float xr[2][4];
        double mk[2][4];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = kb + 16 * b + 4 * g + s;
                xr[b][s] = rok && k < d ? elem<DT>::ld(X, row * ld + k) : 0.0f;
                mk[b][s] = k < d ? mu[k] : 0.0;
            }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t < nt) {
                const int jj = 16 * t + r;
                double ub[2][4];
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int k = kb + 16 * b + 4 * g + s;
                        ub[b][s] = k < d && jj < p ? U[(int64_t)k * p + jj] : 0.0;
                    }
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const double xa = rok ? (double)xr[b][s] - mk[b][s] : 0.0;
                        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, ub[b][s], acc[t], 0, 0, 0);
                    }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (t < nt) {
            const int jj = 16 * t + r;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t rr = row0 + g + 4 * i;
                if (rr < n && jj < p) Z[rr * p + jj] = (float)acc[t][i];
            }
        }
    }
}

template <typename F>
static void pca_by_dtype(int dt, F&& f)
{
    if (dt == KNN_F32) f(std::integral_constant<int, KNN_F32>());
    else if (dt == KNN_BF16) f(std::integral_constant<int, KNN_BF16>());
    else f(std::integral_constant<int, KNN_F16>());
}

}  // namespace knn

using namespace knn;

extern "C" knn_status knn_pca(knn_matrix X, int32_t p, int32_t iters, float* Z, double* components,
                              double* eigenvalues, double* mean, void* stream)
{
    try {
        knn_status r = check_matrix(X, "X");
        if (r != KNN_OK) return r;
        if (!Z) return fail(KNN_EINVAL, "Z is null");
        if (X.n < 2) return fail(KNN_EINVAL, "X.n must be >= 2");
        if (p < 1 || p > X.d) return fail(KNN_EINVAL, "p must satisfy 1 <= p <= d");
        if (p > kPcaMaxP) return fail(KNN_ENOTSUP, "p above 64 is not supported");
        if (iters < 0) return fail(KNN_EINVAL, "iters must be >= 0");
        const int d = X.d;
        if (d > 16384) return fail(KNN_ENOTSUP, "d above 16384 is not supported by the PCA");
        int m = 2 * p > p + 16 ? 2 * p : p + 16;
        if (m > kPcaMaxM) m = kPcaMaxM;
        if (m > d) m = d;
        const int T = m == d ? 0 : (iters > 0 ? iters : 200);
        const int64_t n = X.n;
        const int nch = (int)ceil_div(n, kPcaChunk);
        const int nsum = (int)ceil_div(n, kPcaSumChunk);
        hipStream_t st = (hipStream_t)stream;
        Workspace ws(st, 0);
        double *part, *mu, *C, *V, *W, *U2, *piv, *S, *H, *E, *U, *lam;
        unsigned* bad;
        const int nt = (int)ceil_div(d, kPcaTile);
        int2* tiles;
        if ((r = ws.alloc(&part, (size_t)std::max<int64_t>((int64_t)nch * d * d, (int64_t)nsum * d))) != KNN_OK)
            return r;
        if ((r = ws.alloc(&mu, (size_t)d)) != KNN_OK) return r;
        if ((r = ws.alloc(&C, (size_t)d * d)) != KNN_OK) return r;
        if ((r = ws.alloc(&V, (size_t)d * m)) != KNN_OK) return r;
        if ((r = ws.alloc(&W, (size_t)d * m)) != KNN_OK) return r;
        if ((r = ws.alloc(&U2, (size_t)d * m)) != KNN_OK) return r;
        if ((r = ws.alloc(&piv, (size_t)3 * m)) != KNN_OK) return r;   // pivots, then the Rayleigh sums
        if ((r = ws.alloc(&S, (size_t)m * m)) != KNN_OK) return r;
        if ((r = ws.alloc(&H, (size_t)m * m)) != KNN_OK) return r;
        if ((r = ws.alloc(&E, (size_t)m * m)) != KNN_OK) return r;
        if ((r = ws.alloc(&U, (size_t)d * p)) != KNN_OK) return r;
        if ((r = ws.alloc(&lam, (size_t)p)) != KNN_OK) return r;
        if ((r = ws.alloc(&bad, 1)) != KNN_OK) return r;
        if ((r = ws.alloc(&tiles, (size_t)nt * (nt + 1) / 2)) != KNN_OK) return r;
        // upper-triangle tile list
        std::vector<int2> tl;
        for (int a = 0; a < nt; ++a)
            for (int b = a; b < nt; ++b) tl.push_back(make_int2(a, b));
        KNN_HIP(hipMemcpyAsync(tiles, tl.data(), tl.size() * sizeof(int2), hipMemcpyHostToDevice, st));
        KNN_HIP(hipMemsetAsync(bad, 0, 4, st));
        pca_by_dtype(X.dtype, [&](auto dt) {
            pca_colsum_kernel<decltype(dt)::value><<<dim3((unsigned)ceil_div(d, 256), (unsigned)nsum), 256, 0, st>>>(
                X.data, n, X.ld, d, part);
        });
        pca_mean_kernel<<<(unsigned)ceil_div(d, 256), 256, 0, st>>>(part, nsum, d, n, mu);
        pca_by_dtype(X.dtype, [&](auto dt) {
            pca_gram_kernel<decltype(dt)::value><<<dim3((unsigned)tl.size(), (unsigned)nch), 256, 0, st>>>(
                X.data, n, X.ld, d, mu, tiles, part);
        });
        pca_gram_reduce_kernel<<<(unsigned)ceil_div((int64_t)d * d, 256), 256, 0, st>>>(part, nch, d, n, C);
        KNN_HIP(hipGetLastError());
        // subspace iteration (skipped when the subspace is all of R^d)
        if (m == d) {
            // V = I: the Rayleigh-Ritz matrix is C itself
            pca_identity_kernel<<<(unsigned)ceil_div((int64_t)d * m, 256), 256, 0, st>>>(d, m, V);
        } else {
            pca_init_kernel<<<(unsigned)ceil_div((int64_t)d * m, 256), 256, 0, st>>>(d, m, 0x5CA1AB1Eull, W);
        }
        const dim3 gcols((unsigned)ceil_div(d, 64), (unsigned)ceil_div(m, kPcaCols));
        const dim3 gcv((unsigned)ceil_div(d, 16), (unsigned)ceil_div(m, 16));
        // shift of the shifted passes: 11 (m d + m (m + 1)) u relative to
        // trace(S) >= |W|_2^2, the bound under which a shifted Cholesky-QR
        // is guaranteed to succeed in double precision (Fukaya, Kannan,
        // Nakatsukasa, Yamamoto and Yanagisawa, 2020)
        const double shift = 11.0 * ((double)m * d + (double)m * (m + 1)) * 1.1102230246251565e-16;
        auto cholqr = [&](const double* in, double* out, double sh) {
            pca_gram_small_kernel<<<dim3((unsigned)m, (unsigned)m), 256, 0, st>>>(in, in, d, m, S);
            pca_cholqr_kernel<<<gcols, 256, 0, st>>>(S, in, d, m, out, bad, piv, sh);
        };
        auto cv = [&](const double* in, double alpha, double sh, const double* prev, double* out) {
            pca_cv_kernel<<<gcv, 256, 0, st>>>(C, in, d, m, alpha, sh, prev, out);
        };
        if (m < d) {
            // Chebyshev-filtered subspace iteration.  A round multiplies V by
            // T_q(2 C / b - 1) (three-term recurrence): components with
            // eigenvalues below b stay at 1, one at lambda grows as
            // cosh(q acosh(2 lambda / b - 1)).  b is the smallest Rayleigh quotient
            // of the last round's columns (at most lambda_m); the first two
            // rounds, before there is one, are plain products.
            //  q: the strongest component may outgrow the damped ones by 1e10
            //     per round, so that rounding of the former (1e-16) stays small
            //     against the latter; at most 8, and 1 after a pass whose
            //     smallest pivot (of unit-length columns) shows them dependent
            //     to 1e-4.
            //  Stop: when the p-th quotient's component has grown e^38 more
            //     than the m-th's over the rounds so far (both re-evaluated
            //     from the current quotients): the error against the wanted
            //     span is then below rounding.  Or, from K = 0.35 T products on
            //     (at least min(T, 24)), when it has grown at least as much more
            //     than lambda_{m+1}'s as T power iterations would give, (lambda_p /
            //     lambda_{m+1})^T.  lambda_{m+1} is not known, but lies between the
            //     eigenvalues' sum of squares over their sum outside the block
            //     (C's Frobenius norm and trace less the block's) and the m-th
            //     quotient; where the former is at least that of a spectrum that
            //     goes on with the block's mean spacing, lambda_{m+1} is taken to
            //     be at most eight spacings below the m-th (noise and
            //     power laws: within one; a drop right behind the block fails
            //     the test).
            //     Five values are tried, and the next round's b is the one with
            //     most left to gain.  Above b the logarithm of T_q
            //     rises by q / sqrt(lambda (lambda - b)), that of lambda^q by q / lambda,
            //     so such rounds gain on the power iterations at that value
            //     and above.  T + K products at most.
            // On a 70,000 x 784 set (eigenvalues as i^-1.2, p = 50) 200 power
            // iterations with a pass after each took 21 of the call's 26 ms;
            // 32 products in 12 rounds take 1.5 of 5.2 ms.
            const int K = std::max(std::min(T, 24), (int)std::ceil(0.35 * T));
            std::vector<double> hv((size_t)3 * m), rho((size_t)m);
            double rest = -1.0;   // lower bound of lambda_{m+1}
            std::vector<std::pair<int, double>> rounds;   // (q, b), b = 0: plain
            double b = 0.0;
            int q = 1;
            cholqr(W, V, shift);
            for (int done = 0;;) {
                const bool plain = rounds.size() < 2 || !(b > 0.0);
                const int qq = plain ? 1 : std::min(q, T + K - done);
                const double c = plain ? 0.0 : 0.5 * b;
                // Y_1 = (C V - c V) / c, Y_{k+1} = 2 (C Y_k - c Y_k) / c - Y_{k-1}
                cv(V, plain ? 1.0 : 1.0 / c, c, nullptr, W);
                pca_rayleigh_kernel<<<(unsigned)m, 256, 0, st>>>(V, W, d, m, piv + m);
                double *cur = W, *prev = V;
                for (int k = 1; k < qq; ++k) {
                    double* out = k == 1 ? U2 : prev;
                    cv(cur, 2.0 / c, c, prev, out);
                    prev = cur;
                    cur = out;
                }
                cholqr(cur, V, shift);
                done += qq;
                rounds.push_back({qq, plain ? 0.0 : b});
                if (done >= T + K || (T == 1 && done == 1)) break;
                KNN_HIP(hipMemcpyAsync(hv.data(), piv, (size_t)3 * m * 8, hipMemcpyDeviceToHost, st));
                KNN_HIP(hipStreamSynchronize(st));
                double lo = hv[0];
                for (int k = 0; k < m; ++k) {
                    lo = std::min(lo, hv[k]);
                    const double vv = hv[2 * m + k], r1 = vv > 0.0 ? hv[m + k] / vv : 0.0;
                    rho[k] = plain ? r1 : c * r1 + c;
                }
                std::sort(rho.begin(), rho.end(), [](double x, double y) { return x > y; });
                const double top = rho[0], wanted = rho[p - 1];
                b = rho[m - 1];
                // how much more a component at `wanted` has grown than one at l, as a
                // logarithm (T_q(x) = cosh(q acosh x), at most 1 for x <= 1)
                auto grown = [](double l, int q, double b) {
                    if (!(b > 0.0)) return q * std::log(l);
                    const double y = q * std::acosh(std::max(2.0 * l / b - 1.0, 1.0));
                    return y + std::log1p(std::exp(-2.0 * y)) - std::log(2.0);
                };
                auto gain = [&](double l) {
                    double g = 0.0;
                    for (const auto& rd : rounds)
                        g += grown(wanted, rd.first, rd.second) - grown(l, rd.first, rd.second);
                    return g;
                };
                if (b > 0.0 && gain(b) >= 38.0) break;
                if (done >= K) {
                    if (!(b > 0.0) || !(wanted > 0.0)) break;   // rank below m
                    if (rest < 0.0) {
                        // squared column norms and diagonal of C, and V^T C V
                        std::vector<double> cn((size_t)2 * d), hb((size_t)m * m);
                        pca_rayleigh_kernel<<<(unsigned)d, 256, 0, st>>>(C, C, d, d, U2);
                        pca_diag_kernel<<<(unsigned)ceil_div(d, 256), 256, 0, st>>>(C, d, U2 + d);
                        cv(V, 1.0, 0.0, nullptr, W);
                        pca_gram_small_kernel<<<dim3((unsigned)m, (unsigned)m), 256, 0, st>>>(W, V, d, m, S);
                        KNN_HIP(hipMemcpyAsync(cn.data(), U2, (size_t)2 * d * 8, hipMemcpyDeviceToHost, st));
                        KNN_HIP(hipMemcpyAsync(hb.data(), S, (size_t)m * m * 8, hipMemcpyDeviceToHost, st));
                        KNN_HIP(hipStreamSynchronize(st));
                        double one = 0.0, two = 0.0, all = 0.0;
                        for (int k = 0; k < d; ++k) {
                            all += cn[k];
                            one += cn[d + k];
                        }
                        two = all;
                        for (int k = 0; k < m * m; ++k) two -= hb[k] * hb[k];
                        for (int k = 0; k < m; ++k) one -= hb[k * m + k];
                        // the mean where the squares are lost in rounding
                        rest = two > 1e-12 * all ? two / one : one / (d - m);
                        rest = one > 0.0 ? std::max(rest, one / (d - m)) : 0.0;
                    }
                    const double step = (wanted - b) / (m - p);
                    double l1 = 0.0, l2 = 0.0;
                    for (int k = 1; k <= d - m && b - step * k > 0.0; ++k) {
                        l1 += b - step * k;
                        l2 += (b - step * k) * (b - step * k);
                    }
                    const double goes_on = rest * l1 >= l2 ? b - 8.0 * step : 0.0;
                    const double least = std::min(std::max({rest, goes_on, 1e-16 * top}), b);
                    double most = 1e-9, at = 0.0;
                    for (int i = 0; i < 5; ++i) {
                        const double l = b * std::pow(least / b, 0.25 * i);
                        const double left = std::min(38.0, T * std::log(wanted / l)) - gain(l);
                        if (left > most) {
                            most = left;
                            at = l;
                        }
                    }
                    if (!(at > 0.0)) break;
                    b = at;
                }
                const double x = b > 0.0 ? 2.0 * top / b - 1.0 : 1e300;
                q = x > 1.0 + 1e-9 ? (int)(std::log(1e10) / std::acosh(x)) : kPcaMaxQ;
                q = lo < 1e-8 ? 1 : std::max(1, std::min(q, kPcaMaxQ));
            }
            cholqr(V, W, shift);
            cholqr(W, V, 0.0);
            cholqr(V, W, 0.0);
            std::swap(V, W);
            KNN_HIP(hipGetLastError());
        }
        // Rayleigh-Ritz: H = V^T C V
        cv(V, 1.0, 0.0, nullptr, W);
        pca_gram_small_kernel<<<dim3((unsigned)m, (unsigned)m), 256, 0, st>>>(W, V, d, m, H);
        pca_jacobi_kernel<<<1, kJacThreads, 0, st>>>(H, E, m);
        pca_ritz_kernel<<<(unsigned)p, 256, 0, st>>>(H, E, V, d, m, p, U, lam, m < d ? bad : nullptr);
        pca_by_dtype(X.dtype, [&](auto dt) {
            pca_project_kernel<decltype(dt)::value><<<(unsigned)ceil_div(n, 64), 256, 0, st>>>(
                X.data, n, X.ld, d, mu, U, p, Z);
        });
        KNN_HIP(hipGetLastError());
        if (components) KNN_HIP(hipMemcpyAsync(components, U, (size_t)d * p * 8, hipMemcpyDeviceToDevice, st));
        if (eigenvalues) KNN_HIP(hipMemcpyAsync(eigenvalues, lam, (size_t)p * 8, hipMemcpyDeviceToDevice, st));
        if (mean) KNN_HIP(hipMemcpyAsync(mean, mu, (size_t)d * 8, hipMemcpyDeviceToDevice, st));
        unsigned hb = 0;
        KNN_HIP(hipMemcpyAsync(&hb, bad, 4, hipMemcpyDeviceToHost, st));
        KNN_HIP(hipStreamSynchronize(st));
        if (hb) return fail(KNN_EINVAL, "X has rank below the subspace width");
        return KNN_OK;
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}
