// UMAP membership strengths of a k-NN graph and their fuzzy union
// (McInnes, Healy & Melville 2018): the graph the UMAP-family methods of the
// paper build from the shared k-NN stage (sections "Architecture" and
// "Method Implementations").
//
// For row i with neighbour distances d_1..d_k:
//   rho_i   = the smallest positive d_r (0 if there is none);
//   sigma_i solves sum_r exp(-max(0, d_r - rho_i) / sigma_i) = log2(k); the
//           sum falls from k (sigma -> inf) to c_i = #{r : d_r <= rho_i}
//           (sigma -> 0), so there is a root iff c_i < log2(k), else
//           sigma_i = 0 and the weights take the limit (1 where d_r <= rho_i,
//           0 elsewhere);
//   w_ir    = exp(-max(0, d_r - rho_i) / sigma_i);
// and the symmetric graph W = A + A^T - A o A^T with A[i][idx_ir] = w_ir.
//
// 1. rows:   one thread per row.  sigma is bracketed and found in FP32
//            (safeguarded Newton, v_exp_f32), then polished by Newton steps on
//            the sum in double, whose root it converges to quadratically from
//            the FP32 estimate; the weights are evaluated in double and
//            rounded once.  Each edge e = (i -> j) is keyed by its target j.
// 2. sort:   the edges are sorted by target with a stable LSD radix sort
//            (32-bit keys, the edge number as payload), so the edges into a
//            row form one segment ordered by source: the row's transposed
//            entries, already in column order.  Deterministic whatever the
//            thread order.
// 3. union:  16 (k <= 16) or 32 lanes per row merge its own k entries (ranked
//            by column) with that segment: a column in both gets the
//            probabilistic union a + b - ab (folded in double in the order
//            of the entries' numbers, 2e for (i, j) and 2e' + 1 for the
//            transposed (j, i) of e' = (j -> i)), the others keep their
//            weight; each entry's CSR position follows from the counts of
//            smaller columns on both sides.  A count pass and a scan over
//            the rows give row_ptr, then the emit pass writes the entries.
#include <math.h>

#include "knn_common.hpp"

namespace knn {

constexpr int kFzMaxK = KNN_MAX_K;   // 32: a row's entries fit the lanes of half a wave
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ rows

// n / k for n < 2^31 as (n * mul) >> (32 + shift) (k = 1: n itself), with
// mul = ceil(2^(31 + l) / k), l = ceil(log2 k), shift = l - 1: the rounding of mul
// adds less than 2^l n / (k 2^(31 + l)) < 1 / k.
struct DivK {
    uint32_t k, mul;
    int shift;
};
static DivK div_by(int k)
{
    int l = 0;
    while ((1 << l) < k) ++l;
    return {(uint32_t)k, k > 1 ? (uint32_t)((((uint64_t)1 << (31 + l)) + (uint64_t)k - 1) / (uint64_t)k) : 0u, l - 1};
}
__device__ inline uint32_t div_k(uint32_t n, DivK d) { return d.k == 1u ? n : __umulhi(n, d.mul) >> d.shift; }

// Sum of exp(-x_r / s) (s > 0) in FP32, as exp2 of -x_r * (log2(e) / s); with
// G also that of exp(-x_r / s) x_r.
template <int KM, bool G>
__device__ inline float fz_sum32(const float (&x)[KM], int k, float s, float* g)
{
    const float c = 1.4426950408889634f / s;
    float t = 0.0f, tg = 0.0f;
#pragma unroll
    for (int r = 0; r < KM; ++r) {
        if (r < k) {
            const float e = __builtin_amdgcn_exp2f(-x[r] * c);
            t += e;
            if (G) tg = fmaf(e, x[r], tg);
        }
    }
    if (G) *g = tg;
    return t;
}

// One thread per row; the block's rows pass through LDS both ways, so that
// memory sees whole lines (a row is k floats: straight loads and stores touch
// 64 lines each).  KM: k <= KM.  sigma is bracketed, found by safeguarded
// Newton steps in FP32 (5 to 7 sums; bisection took 25) and polished in
// double until a step is below 1e-6 of it (the next error is its square).
// 1,000,000 x 15: 119 us, bound by the exponentials; 446 with straight loads and
// stores, bisection, and four steps in double always.
template <int KM>
__global__ __launch_bounds__(256) void fuzzy_rows_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ dist, int64_t n, int k, DivK dk,
    float* __restrict__ rho_out, float* __restrict__ sigma_out, float* __restrict__ w_out,
    uint32_t* __restrict__ tgtkey, unsigned* __restrict__ bad)
{
    __shared__ float buf[256 * (KM + 1)];   // row r at r * ks, ks odd
    const int tid = threadIdx.x, ks = k | 1;
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + tid, e0 = i0 * k;
    const int rows = (int)(n - i0 < 256 ? n - i0 : 256), ne = rows * k;
    bool ok = true;
    for (int c = tid; c < ne; c += 256) {
        const uint32_t r = div_k((uint32_t)c, dk);
        buf[r * ks + (c - r * k)] = dist[e0 + c];
        const int32_t j = idx[e0 + c];
        const bool valid = j >= 0 && (int64_t)j < n && (int64_t)j != i0 + r;
        ok = ok && valid;
        // keyed by target; invalid edges sort last (key n)
        tgtkey[e0 + c] = valid ? (uint32_t)j : (uint32_t)n;
    }
    if (!ok) atomicOr(bad, 1u);
    __syncthreads();
    if (tid < rows) {
        float d[KM];
        double p = 0.0;
#pragma unroll
        for (int r = 0; r < KM; ++r) {
            d[r] = r < k ? buf[tid * ks + r] : 0.0f;
            if (r < k && d[r] > 0.0f && (p == 0.0 || (double)d[r] < p)) p = (double)d[r];
        }
        // x_r = max(0, d_r - rho) in double (exact for FP32 inputs), kept as
        // FP32 for the bracket search
        float x[KM];
        int cnt = 0;
        float xmax = 0.0f;
#pragma unroll
        for (int r = 0; r < KM; ++r) {
            const double xd = (double)d[r] - p;
            x[r] = xd > 0.0 ? (float)xd : 0.0f;
            if (r < k && !(xd > 0.0)) ++cnt;
            if (r < k) xmax = fmaxf(xmax, x[r]);
        }
        const double target = log2((double)k);
        double sig = 0.0;
        if ((double)cnt < target) {
            const float t32 = (float)target;
            float lo = 0.0f, hi = xmax, g;
            while (fz_sum32<KM, false>(x, k, hi, nullptr) < t32) hi *= 2.0f;
            float s32 = 0.5f * hi;
            for (int it = 0; it < 40; ++it) {
                if (!(s32 > lo && s32 < hi)) s32 = 0.5f * (lo + hi);
                if (!(s32 > lo && s32 < hi)) break;
                const float f = fz_sum32<KM, true>(x, k, s32, &g) - t32;
                if (f < 0.0f) lo = s32;
                else hi = s32;
                const float step = f * s32 * s32 / g;
                s32 -= step;
                if (fabsf(step) < 4e-7f * s32) break;   // not where both are infinite (g = 0)
            }
            // Newton on f(s) = sum exp(-x_r / s) - log2(k), f'(s) = sum
            // exp(-x_r / s) x_r / s^2, in double
            s32 = fminf(fmaxf(s32, lo), hi);
            double s = s32 > 0.0f && s32 < __builtin_inff() ? (double)s32 : 0.5 * ((double)lo + (double)hi);
            for (int it = 0; it < 4; ++it) {
                double f = -target, gd = 0.0;
#pragma unroll
                for (int r = 0; r < KM; ++r) {
                    if (r < k) {
                        const double xr = fmax((double)d[r] - p, 0.0);
                        const double e = exp(-xr / s);
                        f += e;
                        gd += e * xr;
                    }
                }
                gd /= s * s;
                if (!(gd > 0.0)) break;
                const double ns = s - f / gd;
                if (!(ns > 0.0) || !isfinite(ns)) break;
                const bool last = fabs(ns - s) <= 1e-6 * ns;
                s = ns;
                if (last) break;
            }
            sig = s;
        }
        if (rho_out) rho_out[i] = (float)p;
        if (sigma_out) sigma_out[i] = (float)sig;
#pragma unroll
        for (int r = 0; r < KM; ++r) {
            if (r < k) {
                const double xr = fmax((double)d[r] - p, 0.0);
                buf[tid * ks + r] = sig > 0.0 ? (float)exp(-xr / sig) : (xr == 0.0 ? 1.0f : 0.0f);
            }
        }
    }
    __syncthreads();
    for (int c = tid; c < ne; c += 256) {
        const uint32_t r = div_k((uint32_t)c, dk);
        w_out[e0 + c] = buf[r * ks + (c - r * k)];
    }
}

// ------------------------------------------------------------------ union

// in_ptr[r] = the first sorted position whose target is >= r, r = 0..n.
__global__ __launch_bounds__(256) void fuzzy_inptr_kernel(const uint32_t* __restrict__ key, int64_t m, int64_t n,
                                                          uint32_t* __restrict__ in_ptr)
{
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < m; p += (int64_t)gridDim.x * 256) {
        const int64_t r = key[p], prev = p > 0 ? (int64_t)key[p - 1] : -1;
        for (int64_t rr = prev + 1; rr <= r; ++rr) in_ptr[rr] = (uint32_t)p;
        if (p == m - 1)
            for (int64_t rr = r + 1; rr <= n; ++rr) in_ptr[rr] = (uint32_t)m;
    }
}

// A wave takes 64 / G consecutive rows (k <= G).  Row i's G lanes rank its own
// entries (i, idx_ir) by column and hold them in that order; the transposed
// entries (i, j) of the edges j -> i are the segment [in_ptr[i], in_ptr[i + 1])
// of the sorted edges, in column order, and each own lane finds its place and
// its partner there by bisection.  The count pass (EMIT false) stores the
// union's size in cnt[i] and flags a column repeated in a row's list; the emit
// pass writes the union at row_ptr[i], columns ascending.  Its transposed
// entries are taken 64 at a time over all of the wave's rows (their segments
// follow each other; a hub gets every lane): each finds its place among
// its row's own entries by bisection in LDS.
// 1,000,000 x 15: 121 and 333 us; 734 and 708 with a wave per row and
// every pair of own and transposed entry compared.  Bound by the latency of the
// bisections; the gather of the transposed entries' weights (a line per entry)
// is 75 us of the emit pass, and carrying them through the sort cost 120 there.
template <bool EMIT, int G>
__global__ __launch_bounds__(256) void fuzzy_union_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ w, int k, DivK dk, int64_t n,
    const uint32_t* __restrict__ sorted_e, const uint32_t* __restrict__ in_ptr, uint32_t* __restrict__ cnt,
    const int64_t* __restrict__ row_ptr, int32_t* __restrict__ col_out, float* __restrict__ val_out,
    unsigned* __restrict__ bad)
{
    constexpr int NR = 64 / G;   // rows per wave
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    __shared__ __attribute__((aligned(16))) uint32_t raw_s[4][64];   // own columns as given
    __shared__ uint32_t own_s[4][64];    // own columns ascending
    __shared__ float ow_s[4][64];        // and their weights
    __shared__ uint32_t match_s[4][NR];  // own entries (bits) with a transposed partner
    __shared__ uint32_t seg_s[4][NR + 1];
    __shared__ int64_t base_s[4][NR];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane / G, r = lane % G;
    const int64_t i0 = ((int64_t)blockIdx.x * 4 + wv) * NR, i = i0 + g;
    if (i0 >= n) return;   // the whole wave
    const bool row = i < n;
    // own entries; an invalid one (reported by the rows kernel) takes no part
    const int32_t jj = row && r < k ? idx[i * k + r] : -1;
    const bool given = jj >= 0 && (int64_t)jj < n && (int64_t)jj != i;
    const uint32_t gc = given ? (uint32_t)jj : kNone;
    const float gw = EMIT && given ? w[i * k + r] : 0.0f;
    const uint32_t b = in_ptr[row ? i : n], e = in_ptr[row ? i + 1 : n];
    raw_s[wv][lane] = gc;
    if (r == 0) {
        seg_s[wv][g] = b;
        if (g == NR - 1) seg_s[wv][NR] = e;
        if (EMIT) base_s[wv][g] = row ? row_ptr[i] : 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // place among the row's entries: smaller columns, and equal ones given before
    uint32_t place = 0;
#pragma unroll
    for (int t = 0; t < G; t += 4) {
        const u32x4 c = *(const u32x4*)&raw_s[wv][g * G + t];
#pragma unroll
        for (int q = 0; q < 4; ++q) place += c[q] < gc || (c[q] == gc && t + q < r) ? 1u : 0u;
    }
    own_s[wv][g * G + place] = gc;
    if (EMIT) ow_s[wv][g * G + place] = gw;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint32_t oc = own_s[wv][lane];
    const bool ov = oc != kNone;
    if (!EMIT) {
        const uint32_t prev = r > 0 ? own_s[wv][lane - 1] : kNone;
        if (ballot(ov && prev == oc) && lane == 0) atomicOr(bad, 2u);
    }
    // transposed entries with a smaller column: edges below oc * k
    uint32_t lo = b, hi = ov ? e : b;
    const uint32_t first = oc * dk.k;
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (sorted_e[mid] < first) lo = mid + 1;
        else hi = mid;
    }
    const bool om = ov && lo < e && sorted_e[lo] - first < dk.k;
    const uint64_t below = ~0ull >> (64 - G) << (g * G);   // the row's lanes
    const uint64_t matched = ballot(om) & below;
    if (!EMIT) {
        const uint32_t nown = (uint32_t)popc64(ballot(ov) & below);
        if (row && r == 0) cnt[i] = nown + (e - b) - (uint32_t)popc64(matched);
        return;
    }
    const uint32_t mbits = (uint32_t)(matched >> (g * G));
    if (r == 0) match_s[wv][g] = mbits;
    if (ov) {
        const float ow = ow_s[wv][lane];
        float v = ow;
        if (om) {
            // entry 2e of (i, j) precedes entry 2e' + 1 of (j, i) iff i < j
            const float wm = w[sorted_e[lo]];
            const double x0 = (double)((int64_t)i < (int64_t)oc ? ow : wm), x1 = (double)((int64_t)i < (int64_t)oc ? wm : ow);
            v = (float)(x0 + x1 - x0 * x1);
        }
        const int64_t pos = base_s[wv][g] + r + (lo - b) - popc64(mbits & ((1u << r) - 1u));
        col_out[pos] = (int32_t)oc;
        val_out[pos] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // transposed entries without a partner: their index in the segment plus the
    // unmatched own entries with a smaller column
    const uint32_t pe = seg_s[wv][NR];
    for (uint32_t p = seg_s[wv][0] + lane; p < pe; p += 64) {
        int h = 0;   // its row
#pragma unroll
        for (int q = 1; q < NR; ++q) h += p >= seg_s[wv][q] ? 1 : 0;
        const uint32_t ed = sorted_e[p], ic = div_k(ed, dk);
        const uint32_t* own = own_s[wv] + h * G;
        uint32_t c = 0;   // own entries with a smaller column
#pragma unroll
        for (uint32_t t = G / 2; t > 0; t >>= 1) c += own[c + t - 1] < ic ? t : 0u;
        const uint32_t at = own[c];
        if (at == ic) continue;
        c += at < ic ? 1u : 0u;
        const uint32_t um = c - (uint32_t)popc64(match_s[wv][h] & ((1ull << c) - 1ull));
        const int64_t pos = base_s[wv][h] + (p - seg_s[wv][h]) + um;
        col_out[pos] = (int32_t)ic;
        val_out[pos] = w[ed];
    }
}

// Row counts to row_ptr: per-block sums over 1024 rows, their exclusive scan
// (fuzzy_scan_kernel, one block), then each block's rows.
constexpr int kFzScanRows = 1024;

// Exclusive scan of a[0..m) in place by one block (in order, with a
// carry); a[m] receives the total.
__global__ __launch_bounds__(256) void fuzzy_scan_kernel(uint32_t* __restrict__ a, int64_t m)
{
    __shared__ uint32_t s[256];
    uint32_t carry = 0;
    for (int64_t b0 = 0; b0 < m; b0 += 256) {
        const int64_t b = b0 + threadIdx.x;
        const uint32_t x = b < m ? a[b] : 0u;
        __syncthreads();
        s[threadIdx.x] = x;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const uint32_t y = (int)threadIdx.x >= o ? s[threadIdx.x - o] : 0u;
            __syncthreads();
            s[threadIdx.x] += y;
            __syncthreads();
        }
        if (b < m) a[b] = carry + s[threadIdx.x] - x;
        carry += s[255];
    }
    if (threadIdx.x == 0) a[m] = carry;
}

__global__ __launch_bounds__(256) void fuzzy_block_sum_kernel(const uint32_t* __restrict__ cnt, int64_t n,
                                                              uint32_t* __restrict__ bsum)
{
    __shared__ uint32_t s[4];
    uint32_t t = 0;
    for (int q = 0; q < 4; ++q) {
        const int64_t i = (int64_t)blockIdx.x * kFzScanRows + threadIdx.x * 4 + q;
        t += i < n ? cnt[i] : 0u;
    }
    for (int o = 32; o > 0; o >>= 1) t += shfl_u32(t, (threadIdx.x & 63) ^ o);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) bsum[blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

__global__ __launch_bounds__(256) void fuzzy_rowptr_kernel(const uint32_t* __restrict__ cnt, int64_t n,
                                                           const uint32_t* __restrict__ boff, int64_t nb,
                                                           int64_t* __restrict__ row_ptr)
{
    __shared__ uint32_t s[256];
    uint32_t c[4], t = 0;
    for (int q = 0; q < 4; ++q) {
        const int64_t i = (int64_t)blockIdx.x * kFzScanRows + threadIdx.x * 4 + q;
        c[q] = i < n ? cnt[i] : 0u;
        t += c[q];
    }
    s[threadIdx.x] = t;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint32_t y = (int)threadIdx.x >= o ? s[threadIdx.x - o] : 0u;
        __syncthreads();
        s[threadIdx.x] += y;
        __syncthreads();
    }
    int64_t run = (int64_t)boff[blockIdx.x] + s[threadIdx.x] - t;
    for (int q = 0; q < 4; ++q) {
        const int64_t i = (int64_t)blockIdx.x * kFzScanRows + threadIdx.x * 4 + q;
        if (i < n) row_ptr[i] = run;
        run += c[q];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) row_ptr[n] = boff[nb];
}

static int bits_for(int64_t v)   // bits to hold values 0..v
{
    int b = 1;
    while (b < 32 && ((int64_t)1 << b) <= v) ++b;
    return b;
}

}  // namespace knn

using namespace knn;

extern "C" knn_status knn_fuzzy_graph(const int32_t* knn_idx, const float* knn_dist, int64_t n, int32_t k,
                                      float* rho, float* sigma, float* weights, int64_t* row_ptr,
                                      int32_t* col, float* val, int64_t* nnz, void* stream)
{
    try {
        if (!knn_idx || !knn_dist || !row_ptr || !col || !val || !nnz) return fail(KNN_EINVAL, "null argument");
        if (n < 2 || n >= (int64_t)0x7FFFFFFF) return fail(KNN_EINVAL, "n must satisfy 2 <= n < 2^31 - 1");
        if (k < 1 || (int64_t)k > n - 1) return fail(KNN_EINVAL, "k must satisfy 1 <= k <= n-1");
        if (k > kFzMaxK) return fail(KNN_ENOTSUP, "k above 32 is not supported by the fuzzy graph");
        const int64_t m = n * (int64_t)k;   // edges
        if (2 * m >= ((int64_t)1 << 32)) return fail(KNN_ENOTSUP, "2 n k must be below 2^32");
        hipStream_t st = (hipStream_t)stream;
        Workspace ws(st, 0);
        knn_status r;
        uint32_t *key, *eid, *k1, *v1, *counts, *inptr, *cnt, *bsum;
            unsigned* bad;
        float* w = weights;
        const int64_t nb = ceil_div(n, kFzScanRows);
        if ((r = ws.alloc(&key, (size_t)m)) != KNN_OK) return r;
        if ((r = ws.alloc(&eid, (size_t)m)) != KNN_OK) return r;
        if ((r = ws.alloc(&k1, (size_t)m)) != KNN_OK) return r;
        if ((r = ws.alloc(&v1, (size_t)m)) != KNN_OK) return r;
        if ((r = ws.alloc(&counts, radix_counts_words(m))) != KNN_OK) return r;
        if ((r = ws.alloc(&inptr, (size_t)n + 1)) != KNN_OK) return r;
        if ((r = ws.alloc(&cnt, (size_t)n)) != KNN_OK) return r;
        if ((r = ws.alloc(&bsum, (size_t)nb + 1)) != KNN_OK) return r;
        if ((r = ws.alloc(&bad, 1)) != KNN_OK) return r;
        if (!w && (r = ws.alloc(&w, (size_t)n * k)) != KNN_OK) return r;
        KNN_HIP(hipMemsetAsync(bad, 0, 4, st));
        const DivK dk = div_by(k);
        const unsigned rgrid = (unsigned)ceil_div(n, 256);
        if (k <= 16)
            fuzzy_rows_kernel<16><<<rgrid, 256, 0, st>>>(knn_idx, knn_dist, n, k, dk, rho, sigma, w, key, bad);
        else
            fuzzy_rows_kernel<32><<<rgrid, 256, 0, st>>>(knn_idx, knn_dist, n, k, dk, rho, sigma, w, key, bad);
        KNN_HIP(hipGetLastError());
        // by target (keys <= n: invalid edges last), stably
        if ((r = radix_sort_bits(key, eid, k1, v1, m, counts, st, bits_for(n), 1, true)) != KNN_OK) return r;
        fuzzy_inptr_kernel<<<(unsigned)std::min<int64_t>(ceil_div(m, 256), 8192), 256, 0, st>>>(key, m, n, inptr);
        const unsigned ugrid = (unsigned)ceil_div(n, k <= 16 ? 16 : 8);   // rows per workgroup
        if (k <= 16)
            fuzzy_union_kernel<false, 16><<<ugrid, 256, 0, st>>>(knn_idx, w, k, dk, n, eid, inptr, cnt, nullptr, nullptr,
                                                                 nullptr, bad);
        else
            fuzzy_union_kernel<false, 32><<<ugrid, 256, 0, st>>>(knn_idx, w, k, dk, n, eid, inptr, cnt, nullptr, nullptr,
                                                                 nullptr, bad);
        fuzzy_block_sum_kernel<<<(unsigned)nb, 256, 0, st>>>(cnt, n, bsum);
        fuzzy_scan_kernel<<<1, 256, 0, st>>>(bsum, nb);
        fuzzy_rowptr_kernel<<<(unsigned)nb, 256, 0, st>>>(cnt, n, bsum, nb, row_ptr);
        if (k <= 16)
            fuzzy_union_kernel<true, 16><<<ugrid, 256, 0, st>>>(knn_idx, w, k, dk, n, eid, inptr, cnt, row_ptr, col, val,
                                                                bad);
        else
            fuzzy_union_kernel<true, 32><<<ugrid, 256, 0, st>>>(knn_idx, w, k, dk, n, eid, inptr, cnt, row_ptr, col, val,
                                                                bad);
        KNN_HIP(hipGetLastError());
        unsigned host[2] = {0, 0};
        KNN_HIP(hipMemcpyAsync(&host[0], bad, 4, hipMemcpyDeviceToHost, st));
        KNN_HIP(hipMemcpyAsync(&host[1], bsum + nb, 4, hipMemcpyDeviceToHost, st));
        KNN_HIP(hipStreamSynchronize(st));
        if (host[0] & 1u) return fail(KNN_EINVAL, "knn_idx holds an entry out of range or equal to its row");
        if (host[0] & 2u) return fail(KNN_EINVAL, "knn_idx holds a column twice in one row");
        *nnz = (int64_t)host[1];
        return KNN_OK;
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}
