// Exact k nearest neighbours: tiled MFMA distance GEMM + fused top-k'.
//
// The paper ranks its quality metrics by exact pairwise Euclidean distances
// computed by chunked matrix multiplication, with the norm expansion
// |a - b|^2 = |a|^2 + |b|^2 - 2 a.b of its k-NN section.  Here:
//
//  1. stage: inputs are copied into a zero-padded, 128-byte-aligned layout
//     (pairs of FP16 parts for FP32, or BF16 / FP16 rounded to nearest even),
//     with FP32 row norms and the largest reference norm;
//  2. tile: each workgroup owns 128 query rows and streams 128-row reference
//     tiles through LDS; MFMA (32x32x16 FP16 or BF16 with FP32
//     accumulation; three FP16 products for FP32) produces dot products.  A
//     first pass over a sample of the references gives every query a gate,
//     the second appends the candidates that reach it; under a workspace
//     limit one pass keeps, per query row, the best k' candidates in
//     registers.  The reference set can be split across workgroups to fill
//     the chip; each split keeps its own candidates;
//  3. merge + re-rank: the splits' candidates are merged, the best k' by GEMM
//     distance are re-ranked with FP32 direct differences on the original
//     input values, and the best k kept.  In FP32 precision a row is
//     certified when its k-th re-ranked distance is below the k'-th GEMM
//     distance minus the worst-case GEMM error bound; other rows are
//  4. recomputed exhaustively with direct differences.
#include <math.h>

#include <algorithm>
#include <mutex>

#include "knn_common.hpp"

namespace knn {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kTileRows = 128;    // queries per workgroup and references per tile
constexpr int kListW = 32;        // list width per query row (k' <= 32)

// ------------------------------------------------------------------ stage

// Waves take groups of 4 rows grid-stride: padded copy (zeros beyond d) and
// the squared norm of the stored values: FP64 sums rounded once to FP32
// (within u of the exact norm), or with `aux` FP32 sums (the norms
// NNDescent's distances use).  maxnorm (nullable) receives the
// largest norm's float bits: one atomic per block after an in-block
// reduction.  With `aux`, the last 8 bytes of each row hold two FP32 words
// instead of zeros: the norm and +inf (a per-row value that NNDescent keeps
// current).
template <int DT, int OUT>
__global__ __launch_bounds__(256) void stage_kernel(const void* __restrict__ X, int64_t n, int d,
                                                    int64_t ld, void* __restrict__ Xs, int ldp,
                                                    float* __restrict__ norms,
                                                    unsigned* __restrict__ maxnorm,
                                                    const uint32_t* __restrict__ rowmap, int aux)
{
    constexpr int RB = 4;   // rows per wave and step: their loads are issued together
    __shared__ unsigned smax[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr bool HALF = OUT != KNN_F32;   // 2-byte staged elements
    const int lim = aux ? ldp - (HALF ? 4 : 2) : ldp;
    unsigned wmax = 0;
    for (int64_t row0 = ((int64_t)blockIdx.x * 4 + wv) * RB; row0 < n; row0 += (int64_t)gridDim.x * 4 * RB) {
        int64_t src[RB];
        float s[RB];
        double sd[RB];
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int64_t row = row0 + q < n ? row0 + q : row0;
            src[q] = rowmap ? (int64_t)rowmap[row] : row;
            s[q] = 0.0f;
            sd[q] = 0.0;
        }
        for (int t = lane; t < lim; t += 64) {
            float v[RB];
#pragma unroll
            for (int q = 0; q < RB; ++q) v[q] = t < d ? elem<DT>::ld(X, src[q] * ld + t) : 0.0f;
#pragma unroll
            for (int q = 0; q < RB; ++q) {
                if (row0 + q >= n) continue;
                const int64_t row = row0 + q;
                float x = v[q];
                if constexpr (OUT == KNN_BF16) {
                    uint16_t b = f32_to_bf16_rne(x);
                    ((uint16_t*)Xs)[row * ldp + t] = b;
                    x = __uint_as_float((uint32_t)b << 16);
                } else if constexpr (OUT == KNN_F16) {
                    const _Float16 hv = (_Float16)x;   // round to nearest even
                    ((_Float16*)Xs)[row * ldp + t] = hv;
                    x = (float)hv;
                } else {
                    ((float*)Xs)[row * ldp + t] = x;
                }
                if (aux)
                    s[q] = fmaf(x, x, s[q]);
                else
                    sd[q] = fma((double)x, (double)x, sd[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            if (aux) {
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) s[q] += xor_f32(s[q], o);
            } else {
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) {
                    const uint64_t b = (uint64_t)__double_as_longlong(sd[q]);
                    const uint64_t y = ((uint64_t)xor_u32((uint32_t)(b >> 32), o) << 32) | xor_u32((uint32_t)b, o);
                    sd[q] += __longlong_as_double((long long)y);
                }
                s[q] = (float)sd[q];
            }
        }
#pragma unroll
        for (int q = 0; q < RB; ++q) {
            const int64_t row = row0 + q;
            if (row >= n) break;
            if (lane == 0) {
                norms[row] = s[q];
                if (aux) {
                    float* a = (float*)((char*)Xs + (row + 1) * (int64_t)ldp * (HALF ? 2 : 4)) - 2;
                    a[0] = s[q];
                    a[1] = __builtin_inff();
                }
            }
            const unsigned u = __float_as_uint(s[q]);
            wmax = u > wmax ? u : wmax;
        }
    }
    if (maxnorm) {
        if (lane == 0) smax[wv] = wmax;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned m = smax[0];
            for (int w = 1; w < 4; ++w) m = smax[w] > m ? smax[w] : m;
            atomicMax(maxnorm, m);
        }
    }
}

// Staging for the FP32 Gram.  A row is kept as two FP16 parts, x s = hi + lo
// with s a power of two (below): hi = x s rounded to FP16 (11 bits), lo = the
// remainder rounded to FP16, so hi + lo holds x s to 2^-22 relative (or
// 2^-25 absolute, for elements 2^-14 below the scale).  Three FP16 MFMA
// products (hi hi, hi lo, lo hi; FP32 accumulation) then give the dot product
// in a fifth of the FP32 MFMA's matrix cycles, with smaller errors than its
// (three sums of 16 products round less often than eight of two: split_err).
// Self search, FP32 MFMA -> split: 70,000 x 784 70.9 -> 48.0 ms (160 TFLOP/s
// of distances); 10,000 queries x 1M x 50 21.3 -> 9.3 ms.
// 32 elements take 64 bytes of hi, then 64 of lo.
constexpr int KNN_SPLIT = 3;   // staged element kind

// The scale of a matrix whose largest squared row norm has the float bits
// `mx`: a power of two that brings the largest norm to at most 2^13, so that
// no element overflows FP16 and sums of products stay far from FP32's range.
// Exponents stop at +-63 (products of two scales stay finite); norms^2 below
// 2^-100, which would need more, are reported by split_range.
__device__ inline float split_scale(unsigned mx)
{
    const int e = (int)(mx >> 23) - 127;            // norm^2 < 2^(e + 1)
    int k = 13 - ((e + 2) >> 1);                     // norm < 2^ceil((e + 1) / 2)
    k = k > 63 ? 63 : (k < -63 ? -63 : k);
    return mx == 0u ? 1.0f : __uint_as_float((unsigned)(k + 127) << 23);
}
__device__ inline bool split_range(unsigned mx) { return mx == 0u || (mx >> 23) >= 127u - 100u; }

// The queries' scale goes by the largest norm up to 2^14 times the references':
// one query far outside would take the others' parts below FP16's range.
// Beyond that (split_far) elements are cut off at FP16's largest value and the
// row is searched directly.
constexpr unsigned kSplitFar = 28u << 23;   // 2^28 in squared norms
__device__ inline float query_scale(unsigned qmx, unsigned rmx) { return split_scale(min(qmx, rmx + kSplitFar)); }
__device__ inline bool split_far(float qn, unsigned rmx) { return __float_as_uint(qn) > rmx + kSplitFar; }

// Squared row norms of X (FP64 sums rounded once to FP32) and the largest
// one's bits: 16 lanes per row.
template <int DT>
__global__ __launch_bounds__(256) void norm_kernel(const void* __restrict__ X, int64_t n, int d, int64_t ld,
                                                   float* __restrict__ norms, unsigned* __restrict__ maxnorm)
{
    __shared__ unsigned smax[4];
    const int g = threadIdx.x & 15;
    unsigned wmax = 0;
    for (int64_t r0 = (int64_t)blockIdx.x * 32; r0 < n; r0 += (int64_t)gridDim.x * 32) {
        // two rows per group, their loads together
        const int64_t ra = r0 + (threadIdx.x >> 4), rb = ra + 16;
        const int64_t oa = (ra < n ? ra : n - 1) * ld, ob = (rb < n ? rb : n - 1) * ld;
        double sa = 0.0, sb = 0.0;
#pragma unroll 4
        for (int t = g; t < d; t += 16) {
            const double xa = (double)elem<DT>::ld(X, oa + t), xb = (double)elem<DT>::ld(X, ob + t);
            sa = fma(xa, xa, sa);
            sb = fma(xb, xb, sb);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            sa += __longlong_as_double((long long)shfl_xor_u64((uint64_t)__double_as_longlong(sa), o));
            sb += __longlong_as_double((long long)shfl_xor_u64((uint64_t)__double_as_longlong(sb), o));
        }
        const float fa = (float)sa, fb = (float)sb;
        if (g == 0 && ra < n) norms[ra] = fa;
        if (g == 0 && rb < n) norms[rb] = fb;
        const unsigned ua = __float_as_uint(fa), ub = __float_as_uint(fb);
        wmax = ua > wmax ? ua : wmax;
        wmax = ub > wmax ? ub : wmax;
    }
#pragma unroll
    for (int o = 32; o >= 16; o >>= 1) {
        const unsigned y = xor_u32(wmax, o);
        wmax = y > wmax ? y : wmax;
    }
    if ((threadIdx.x & 63) == 0) smax[threadIdx.x >> 6] = wmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned m = smax[0];
        for (int w = 1; w < 4; ++w) m = smax[w] > m ? smax[w] : m;
        atomicMax(maxnorm, m);
    }
}

// The staged rows: thread = 8 elements of a row (16 bytes of hi and of lo),
// zeros beyond d.  OUT = KNN_SPLIT, or KNN_F16 (hi only: 16-bit inputs, whose
// values FP16 holds exactly up to the 2^-25 above).  ldp: elements, a
// multiple of 32 (KNN_SPLIT) or 64.  rmax (nullable): X are queries, of
// references with this largest norm.
template <int DT, int OUT>
__global__ __launch_bounds__(256) void split_kernel(const void* __restrict__ X, int64_t n, int d, int64_t ld,
                                                    _Float16* __restrict__ Xs, int ldp,
                                                    const unsigned* __restrict__ maxnorm,
                                                    const unsigned* __restrict__ rmax)
{
    const float sc = rmax ? query_scale(*maxnorm, *rmax) : split_scale(*maxnorm);
    const int per = ldp / 8;
    const int64_t total = n * per;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256) {
        const int64_t row = q / per;
        const int t0 = (int)(q % per) * 8;
        _Float16 hi[8], lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x = t0 + e < d ? elem<DT>::ld(X, row * ld + t0 + e) * sc : 0.0f;
            x = fminf(fmaxf(x, -65504.0f), 65504.0f);
            hi[e] = (_Float16)x;
            lo[e] = (_Float16)(x - (float)hi[e]);
        }
        if (OUT == KNN_SPLIT) {
            _Float16* o = Xs + row * (2 * (int64_t)ldp) + (t0 / 32) * 64 + t0 % 32;
            *(uint4*)o = *(const uint4*)hi;
            *(uint4*)(o + 32) = *(const uint4*)lo;
        } else {
            *(uint4*)(Xs + row * (int64_t)ldp + t0) = *(const uint4*)hi;
        }
    }
}

// ------------------------------------------------------------------ tile

// Tile geometry per staged element kind (KNN_BF16, KNN_F16, KNN_SPLIT): values
// per K chunk (128 bytes per row), their LDS row stride (144 bytes), and the
// longest query rows that stay in LDS, with their stride.
template <int OUT>
struct TileCfg;
template <>
struct TileCfg<KNN_BF16> {
    using E = uint16_t;
    static constexpr int KC = 64;
    static constexpr int LROW = 72;
    static constexpr int AMAX = 64;
    static constexpr int AROW = 72;
};
template <>
struct TileCfg<KNN_F16> : TileCfg<KNN_BF16> {};
// split rows: a chunk is 32 elements, 32 hi then 32 lo values
template <>
struct TileCfg<KNN_SPLIT> : TileCfg<KNN_BF16> {
    static constexpr int AMAX = 128;
    static constexpr int AROW = 136;
};

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Output D of a 32x32 MFMA: lane l, accumulator v holds row
// 8*(v/4) + 4*(l/32) + v%4 and column l%32 of the 32x32 block.
__device__ inline int mfma_row(int v, int half) { return 8 * (v >> 2) + 4 * half + (v & 3); }

// Adds the keys of the lanes in `m` (lanes 0..31 for the list held by lanes
// 0..31, lanes 32..63 for the one held by lanes 32..63) to the two sorted
// 32-key lists, keeping each list's 32 smallest.  A few keys are inserted one
// at a time per half: lanes whose entry exceeds the key move up one place and
// the first of them takes the key.  Many keys are sorted and merged by
// bitonic networks.  Both routes give the same list.
__device__ inline uint64_t list_add(uint64_t list, uint64_t key, uint64_t m, int lane)
{
    uint32_t m0 = (uint32_t)m, m1 = (uint32_t)(m >> 32);
    if (__builtin_popcount(m0) > 3 || __builtin_popcount(m1) > 3) {
        const uint64_t ck = seg_sort<32>(key);
        return seg_merge_sorted<32>(list, ck);
    }
    const bool hi = lane >= 32, first = (lane & 31) == 0;
    while (m0 | m1) {
        const uint64_t x0 = m0 ? bcast_u64(key, __builtin_ctz(m0)) : kEmptyCand;
        const uint64_t x1 = m1 ? bcast_u64(key, 32 + __builtin_ctz(m1)) : kEmptyCand;
        const uint64_t x = hi ? x1 : x0;
        // entries above x move up one place and the first of them takes x:
        // with the list ascending that is min(entry, max(entry below, x))
        const uint64_t up = shift_up_u64(list);   // by every lane: a masked lane's value would not arrive
        const uint64_t below = first ? 0ull : up;
        list = umin64(list, umax64(below, x));
        m0 &= m0 - 1u;
        m1 &= m1 - 1u;
    }
    return list;
}

// Rows of one pipeline step, loaded into registers: this thread's four
// 16-byte pieces of the 128 reference rows' chunk k0 (and of the query rows'
// when they stream), and the reference norm of tile row tid % 128.  Piece i is bytes 16 (tid % 8) of row 32 i + tid / 8, so the 64 lanes
// of a load read eight whole 128-byte lines.  Rows past the end, and a tile
// past it (the step after the last), read the last row.
struct StepRegs {
    uint4 b0, b1, b2, b3, a0, a1, a2, a3;   // named, not arrays: arrays were left in scratch memory
    float rn;
};

template <typename E, bool ARES>
__device__ inline void load_step(StepRegs& x, const E* Qb, int qlast, const E* Re, int64_t rt, int64_t rend,
                                 int k0, int ldp, const float* rn, int tid)
{
    const int r0 = tid >> 3, col = (tid & 7) * 16;
    rt = rt < rend ? rt : rend - 1;
    const uint32_t rowb = (uint32_t)ldp * (uint32_t)sizeof(E);
    const char* rb = (const char*)(Re + rt * ldp + k0);
    const int rlast = rend - rt > kTileRows ? kTileRows - 1 : (int)(rend - rt) - 1;
    auto at = [&](const char* base, int r, int last) {
        return *(const uint4*)(base + ((uint32_t)(r < last ? r : last) * rowb + (uint32_t)col));
    };
    x.b0 = at(rb, r0, rlast);
    x.b1 = at(rb, r0 + 32, rlast);
    x.b2 = at(rb, r0 + 64, rlast);
    x.b3 = at(rb, r0 + 96, rlast);
    if (!ARES) {
        const char* qb = (const char*)(Qb + k0);
        x.a0 = at(qb, r0, qlast);
        x.a1 = at(qb, r0 + 32, qlast);
        x.a2 = at(qb, r0 + 64, qlast);
        x.a3 = at(qb, r0 + 96, qlast);
    }
    // without a branch: one would hold copies of the pieces, and waits for them
    const int nr = (tid & (kTileRows - 1)) < rlast ? (tid & (kTileRows - 1)) : rlast;
    x.rn = rn[rt + nr];
}

// The query rows' whole length (at most AMAX elements) into LDS once.
template <typename E, int AROW>
__device__ inline void load_queries(E* As, const E* Qb, int qlast, int ldp, int tid)
{
    const int per = ldp * (int)sizeof(E) / 16;   // 16-byte pieces per row
    for (int e = tid; e < kTileRows * per; e += 256) {
        const int r = e / per, col = e % per;
        const int q = r < qlast ? r : qlast;
        *(uint4*)((char*)(As + r * AROW) + 16 * col) = *(const uint4*)((const char*)(Qb + (int64_t)q * ldp) + 16 * col);
    }
}

// All K chunks of reference tile rt (rows rt .. rt + 127, clamped to rend)
// against the workgroup's 128 query rows: wave w's four 32x32 accumulators
// (query rows 32w + .., reference columns 32b + ..) are returned in acc.
// Each step stores the registers loaded by the previous one into LDS and
// issues the loads of the next step (the next tile's first chunk, at rnext or
// rt + 128, after the last chunk), so the loads of a step overlap the MFMAs of the one before.
// With ARES the query rows are already in As (row stride AROW).
// INIT: what the sums start from.  kFromZero; kByColumn: minus half the
// column's squared norm times the scales (hsc), so that a sum is the score
// q.r - |r|^2 / 2 the gate tests; kTransposed: the same with the operands
// swapped (rows = references, columns = queries: a lane's 16 sums belong to
// one query).  Scores of references past rend are -inf.
// kSegmented: operands swapped, from zero, the sums of every kSegChunks chunks
// formed apart and then added: additions then round sums no larger than their
// segment's |q_s||r_s|, which add up to |q||r| at most, so the bound counts one
// segment's instructions instead of all (rank_tile_kernel).
enum { kFromZero = 0, kByColumn = 1, kTransposed = 2, kSegmented = 3 };
constexpr int kSegChunks = 4;

template <int OUT, bool ARES, int INIT = kFromZero>
__device__ __attribute__((always_inline)) inline void tile_gemm(
    StepRegs& nx, f32x16 (&acc)[4], typename TileCfg<OUT>::E* As, typename TileCfg<OUT>::E* Bs, float* srn,
    const typename TileCfg<OUT>::E* Qb, int qlast, const typename TileCfg<OUT>::E* Re, int64_t rt, int64_t rend, int ldp, const float* rn, int tid, int w, int h, int c, float hsc = 0.5f, int64_t rnext = -1)
{
    using C = TileCfg<OUT>;
    using E = typename C::E;
    constexpr int KC = C::KC, LROW = C::LROW, PER = KC / 2;
    constexpr int AROW = ARES ? C::AROW : LROW;
    constexpr int NV = PER * (int)sizeof(E) / 16;   // 16-byte loads per thread and chunk
    static_assert(NV == 4, "four 16-byte pieces per thread and chunk");
    const int sr = tid >> 3, scol = (tid & 7) * 16;   // staging: see load_step
    constexpr bool SWAP = INIT == kTransposed || INIT == kSegmented;
    if (INIT == kFromZero || INIT == kSegmented) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;
    }
    f32x16 seg[4];   // the current segment's sums
    int segc = 0;
    if (INIT == kSegmented) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) seg[b][v] = 0.0f;
    }

    for (int k0 = 0; k0 < ldp; k0 += KC) {
        __syncthreads();   // the previous step's LDS reads are done
        {
            char* bd = (char*)(Bs + sr * LROW) + scol;
            constexpr int RS = 32 * LROW * (int)sizeof(E);
            *(uint4*)bd = nx.b0;
            *(uint4*)(bd + RS) = nx.b1;
            *(uint4*)(bd + 2 * RS) = nx.b2;
            *(uint4*)(bd + 3 * RS) = nx.b3;
            if (!ARES) {
                char* ad = (char*)(As + sr * LROW) + scol;
                *(uint4*)ad = nx.a0;
                *(uint4*)(ad + RS) = nx.a1;
                *(uint4*)(ad + 2 * RS) = nx.a2;
                *(uint4*)(ad + 3 * RS) = nx.a3;
            }
            if (k0 == 0 && tid < kTileRows)
                srn[tid] = rt + tid < rend ? nx.rn : (INIT == kFromZero ? 0.0f : __builtin_inff());
        }
        __syncthreads();
        if (INIT == kByColumn && k0 == 0) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float i0 = -hsc * srn[b * 32 + c];
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][v] = i0;
            }
        }
        if (INIT == kTransposed && k0 == 0) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    const f32x4 x = *(const f32x4*)&srn[b * 32 + 8 * v4 + 4 * h];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[b][4 * v4 + e] = -hsc * x[e];
                }
        }
        // the next step's rows are in flight during this step's arithmetic
        {
            const bool last = k0 + KC >= ldp;
            load_step<E, ARES>(nx, Qb, qlast, Re, last ? (rnext >= 0 ? rnext : rt + kTileRows) : rt, rend, last ? 0 : k0 + KC, ldp, rn, tid);
            __builtin_amdgcn_sched_barrier(0);   // or the scheduler sinks the loads below the arithmetic
        }
        // K permutation: half h of the wave supplies chunk columns
        // h*PER .. h*PER+PER-1, the same for A and B, so every column
        // enters the dot product exactly once.
        // (split rows: columns h * 16 .. + 15 of the chunk's 32, pieces 0 and
        // 1 their hi values, 2 and 3 their lo values)
        constexpr int HP = OUT == KNN_SPLIT ? PER / 2 : PER;
        const uint4* ap = (const uint4*)(As + (w * 32 + c) * AROW + (ARES ? k0 : 0) + h * HP);
        uint4 a4[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) a4[i] = ap[OUT == KNN_SPLIT && i >= 2 ? i + 2 : i];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint4* bp = (const uint4*)(Bs + (b * 32 + c) * LROW + h * HP);
            uint4 b4[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) b4[i] = bp[OUT == KNN_SPLIT && i >= 2 ? i + 2 : i];
            if constexpr (OUT == KNN_SPLIT) {
                f32x16 x = INIT == kSegmented ? seg[b] : acc[b];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const f16x8 ah = __builtin_bit_cast(f16x8, a4[i]), al = __builtin_bit_cast(f16x8, a4[i + 2]);
                    const f16x8 bh = __builtin_bit_cast(f16x8, b4[i]), bl = __builtin_bit_cast(f16x8, b4[i + 2]);
                    x = __builtin_amdgcn_mfma_f32_32x32x16_f16(SWAP ? bl : ah, SWAP ? ah : bl, x, 0, 0, 0);
                    x = __builtin_amdgcn_mfma_f32_32x32x16_f16(SWAP ? bh : al, SWAP ? al : bh, x, 0, 0, 0);
                    x = __builtin_amdgcn_mfma_f32_32x32x16_f16(SWAP ? bh : ah, SWAP ? ah : bh, x, 0, 0, 0);
                }
                if (INIT == kSegmented) seg[b] = x;
                else acc[b] = x;
            } else if constexpr (OUT == KNN_BF16) {
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const bf16x8 av = __builtin_bit_cast(bf16x8, INIT == kTransposed ? b4[i] : a4[i]);
                    const bf16x8 bv = __builtin_bit_cast(bf16x8, INIT == kTransposed ? a4[i] : b4[i]);
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[b], 0, 0, 0);
                }
            } else if constexpr (OUT == KNN_F16) {
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const f16x8 av = __builtin_bit_cast(f16x8, INIT == kTransposed ? b4[i] : a4[i]);
                    const f16x8 bv = __builtin_bit_cast(f16x8, INIT == kTransposed ? a4[i] : b4[i]);
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, acc[b], 0, 0, 0);
                }
            }
        }
        if (INIT == kSegmented) {
            segc = segc + 1 == kSegChunks ? 0 : segc + 1;
            if (segc == 0 || k0 + KC >= ldp) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        acc[b][v] += seg[b][v];
                        seg[b][v] = 0.0f;
                    }
            }
        }
    }
}

// One workgroup (4 waves) owns 128 query rows and streams the reference
// rows [rbeg, rend) of its split in 128-row tiles, K chunk by K chunk.  The
// sequence of (tile, chunk) steps is software-pipelined: the global loads of
// step t+1 are issued into registers before step t's MFMAs and epilogue run
// and are written to LDS at the top of step t+1, so HBM/L2 latency overlaps
// the arithmetic.  With ARES (row length ldp <= AMAX) the query rows are
// loaded into LDS once and only reference rows stream.  Wave w computes
// query rows 32w..32w+31 against the tile's 128 references (four 32x32
// MFMA blocks).
template <int OUT, bool ARES>
__global__ __launch_bounds__(256, 2) void exact_tile_kernel(
    const void* __restrict__ Qs, const float* __restrict__ qn, int64_t nq,
    const void* __restrict__ Rs, const float* __restrict__ rn, int64_t nr, int ldp,
    const int32_t* __restrict__ q_self, int self_mode, int64_t self_base, int kp, int64_t split_len, int S,
    const unsigned* __restrict__ rmax_bits, const unsigned* __restrict__ qmax_bits, uint64_t* __restrict__ part)
{
    constexpr int INIT = ARES ? kByColumn : kFromZero;
    using C = TileCfg<OUT>;
    using E = typename C::E;
    constexpr int KC = C::KC, LROW = C::LROW, PER = KC / 2;
    constexpr int AROW = ARES ? C::AROW : LROW;
    constexpr int NV = PER * (int)sizeof(E) / 16;   // 16-byte loads per thread and chunk
    __shared__ __attribute__((aligned(16))) E As[kTileRows * AROW];
    __shared__ __attribute__((aligned(16))) E Bs[kTileRows * LROW];
    __shared__ float srn[kTileRows];
    __shared__ float sqn[kTileRows];
    __shared__ int32_t sself[kTileRows];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, c = lane & 31;
    const int64_t q0 = (int64_t)blockIdx.x * kTileRows;
    const int s = blockIdx.y;
    const int64_t rbeg = (int64_t)s * split_len;
    const int64_t rend = rbeg + split_len < nr ? rbeg + split_len : nr;

    if (tid < kTileRows) {
        const int64_t qr = q0 + tid;
        sqn[tid] = qr < nq ? qn[qr] : 0.0f;
        sself[tid] = qr >= nq ? -1 : (self_mode == 1 ? (int32_t)(self_base + qr) : (self_mode == 2 ? q_self[qr] : -1));
    }
    // Per-row lists of this lane's 16 accumulator rows and their gates.
    // A candidate enters a list when d2 = |q|^2 + |r|^2 - 2 q.r <= thr (the
    // list's k'-th distance).  The gate tests the equivalent
    // q.r - |r|^2/2 >= (|q|^2 - thr)/2 with two operations per element;
    // lim is lowered by a slack that covers the FP32 rounding of both forms
    // (8u (|q|^2 + thr + max|r|^2)), so every candidate the exact test
    // accepts passes the gate, and the exact test decides.  Rows past nq
    // get lim = +inf and never pass.
    // Scaled rows (qmax_bits not null) leave the accumulators and the gate in
    // units of both scales, powers of two, so nothing is rounded by them.
    const float rmax = __uint_as_float(*rmax_bits);
    const float scq = qmax_bits ? query_scale(*qmax_bits, *rmax_bits) : 1.0f, scr = qmax_bits ? split_scale(*rmax_bits) : 1.0f;
    const float sc = scq * scr, m2 = -2.0f / sc, hsc = 0.5f * sc;
    uint64_t list[16];
    float lim[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        list[v] = kEmptyList;
        const int64_t row = q0 + w * 32 + mfma_row(v, h);
        lim[v] = row >= nq ? __builtin_inff() : -__builtin_inff();
    }

    const E* Qb = (const E*)Qs + q0 * ldp;
    const E* Re = (const E*)Rs;
    const int qlast = nq - q0 > kTileRows ? kTileRows - 1 : (int)(nq - q0) - 1;
    if (ARES) load_queries<E, AROW>(As, Qb, qlast, ldp, tid);

    // prologue: the first step's rows (addresses are clamped to valid rows,
    // so a load past the split's end is harmless)
    StepRegs nx;
    load_step<E, ARES>(nx, Qb, qlast, Re, rbeg, rend, 0, ldp, rn, tid);
    for (int64_t rt = rbeg; rt < rend; rt += kTileRows) {
        f32x16 acc[4];
        tile_gemm<OUT, ARES, INIT>(nx, acc, As, Bs, srn, Qb, qlast, Re, rt, rend, ldp, rn, tid, w, h, c, hsc);

        // epilogue: distances, threshold gate, list updates
        for (int blk = 0; blk < 4; ++blk) {
            const f32x16 cur = blk == 0 ? acc[0] : (blk == 1 ? acc[1] : (blk == 2 ? acc[2] : acc[3]));
            const float rnj = srn[blk * 32 + c];
            const float hr = INIT == kByColumn ? 0.0f : hsc * rnj;
            // gate all 16 rows first: one branch per block when nothing passes
            uint64_t gm[16], any = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                gm[v] = ballot((INIT == kByColumn ? cur[v] : cur[v] - hr) >= lim[v]);
                any |= gm[v];
            }
            if (!any) continue;
            const int32_t j = (int32_t)rt + blk * 32 + c;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if (gm[v]) {
                    // exact test; the list's current k'-th distance is the threshold
                    const int lr = w * 32 + mfma_row(v, h);
                    const float sq = sqn[lr];
                    const uint64_t t0 = bcast_u64(list[v], kp - 1), t1 = bcast_u64(list[v], 32 + kp - 1);
                    const float thr = key_d2(h ? t1 : t0);
                    float d2 = fmaf(m2, cur[v], INIT == kByColumn ? sq : sq + rnj);
                    d2 = d2 > 0.0f ? d2 : 0.0f;
                    const bool ok = j < (int32_t)rend && j != sself[lr] && d2 <= thr && lim[v] < __builtin_inff();
                    const uint64_t okm = ballot(ok);
                    if (okm) {
                        const uint64_t ck = ok ? make_key(d2, (uint32_t)j) : kEmptyCand;
                        list[v] = list_add(list[v], ck, okm, lane);
                        const uint64_t u0 = bcast_u64(list[v], kp - 1), u1 = bcast_u64(list[v], 32 + kp - 1);
                        const float t = key_d2(h ? u1 : u0);
                        const float nl = (0.5f * (sq - t) - 4.76837158e-07f * (sq + t + rmax)) * sc;   // 8u = 2^-21
                        lim[v] = lim[v] < __builtin_inff() ? nl : lim[v];
                    }
                }
            }
        }
    }

#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int64_t row = q0 + w * 32 + mfma_row(v, h);
        if (row < nq) part[(row * S + s) * kListW + c] = list[v];
    }
}

// Descending list of 32 values in registers; x enters through one max and 31
// medians (entry q becomes the median of entries q - 1, q and x).
__device__ inline void top_insert(float (&t)[kListW], float x)
{
    float up = t[0];
    t[0] = fmaxf(up, x);
#pragma unroll
    for (int q = 1; q < kListW; ++q) {
        const float old = t[q];
        t[q] = __builtin_amdgcn_fmed3f(up, old, x);
        up = old;
    }
}

// Without a workspace limit the search takes the gated route: a gate per
// query first, then one pass that only appends what reaches it.  Keeping sorted
// lists in the tile pass (exact_tile_kernel) costs kp (1 + ln(len / kp))
// insertions per row and split, and the 16 unrolled copies of the insertion
// are more code than the instruction cache holds, so each waits for its code:
// 20,011 x 50 in FP16 took 1,101 us, the same products without insertions 122.
// The gated route takes 100 to 130 us for each of its two passes there.
// Whole calls, lists -> gated (MI355X): 5,000 x 50 FP32 420 -> 138 us;
// 20,011 x 50 FP16 1,200 -> 363 us; 100,000 x 50 FP32 12.4 -> 6.5 ms; 10,000
// queries x 1M x 50 FP32 7.2 -> 5.1 ms; 20,000 x 128 FP32 1,210 -> 660 us;
// 70,000 x 784 BF16 17.4 -> 13.8 ms, FP32 28.1 -> 27.8 ms.
//
// Gate.  The pass forms the scores s = q.r - |r|^2 / 2 for ntiles tiles spread
// evenly over the references (tile i at row 128 floor(i all / ntiles); workgroup
// (query block, p) takes tiles p, p + P, ...) with the operands swapped, so
// that a lane holds 16 references of one query per block: the best score of
// each group of 64 references is a max over registers, and the lane keeps the
// best 32 group scores.  The kp-th best of a query's groups is reached by kp
// different references, so a gate at that score, lowered by twice the
// scores' error bound, lets the kp nearest pass.  With g groups it lies near
// the sample's x-th score, g (1 - exp(-x / g)) = kp; groups are 16 references
// up to 48 tiles and four up to 4, so that there are at least 32 of them.  In a self
// search the tile of the queries themselves stands in for the sample's next
// one, in groups of four: where neighbours follow each other (rows sorted by
// position or time) groups are near-copies, and without it 30 of them
// let thousands of references pass (20,000 x 300 along a curve, BF16: 7.15 ms,
// 1.11 with it).
// gtop[(row * P + p) * 32 ..]: the workgroup's best group scores, descending.
template <int OUT, bool ARES>
__global__ __launch_bounds__(256, 2) void exact_gate_kernel(
    const void* __restrict__ Qs, int64_t nq, const void* __restrict__ Rs, const float* __restrict__ rn, int64_t nr,
    int ldp, const int32_t* __restrict__ q_self, int self_mode, int64_t self_base, int ntiles,
    const unsigned* __restrict__ rmax_bits, const unsigned* __restrict__ qmax_bits, float* __restrict__ gtop)
{
    using C = TileCfg<OUT>;
    using E = typename C::E;
    constexpr int LROW = C::LROW, AROW = ARES ? C::AROW : LROW;
    __shared__ __attribute__((aligned(16))) E As[kTileRows * AROW];
    __shared__ __attribute__((aligned(16))) E Bs[kTileRows * LROW];
    __shared__ __attribute__((aligned(16))) float srn[kTileRows];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, c = lane & 31;
    const int64_t q0 = (int64_t)blockIdx.x * kTileRows;
    const int p = blockIdx.y, P = gridDim.y;
    const float hsc = 0.5f * (qmax_bits ? query_scale(*qmax_bits, *rmax_bits) * split_scale(*rmax_bits) : 1.0f);
    const int64_t qr = q0 + w * 32 + c;   // this lane's query
    const int64_t self = qr >= nq ? -1 : (self_mode == 1 ? self_base + qr : (self_mode == 2 ? (int64_t)q_self[qr] : -1));
    const E* Qb = (const E*)Qs + q0 * ldp;
    const E* Re = (const E*)Rs;
    const int qlast = nq - q0 > kTileRows ? kTileRows - 1 : (int)(nq - q0) - 1;
    if (ARES) load_queries<E, AROW>(As, Qb, qlast, ldp, tid);
    float top[kListW];
#pragma unroll
    for (int q = 0; q < kListW; ++q) top[q] = -__builtin_inff();
    const int64_t all = ceil_div(nr, kTileRows);
    StepRegs nx;
    // the queries' own tile, or for those of a last tile in part the one before
    const int64_t own = self_mode == 1 ? min((self_base + q0) / kTileRows, nr / kTileRows - 1) : -1;
    const auto row_of = [&](int i) {
        const int64_t t = (int64_t)i * all / ntiles;
        return (own >= t && own < (int64_t)(i + 1) * all / ntiles ? own : t) * kTileRows;
    };
    int64_t rt = row_of(p), rnext;
    load_step<E, ARES>(nx, Qb, qlast, Re, rt, nr, 0, ldp, rn, tid);
    for (int i = p; i < ntiles; i += P, rt = rnext) {
        rnext = row_of(i + P);
        f32x16 acc[4];
        tile_gemm<OUT, ARES, kTransposed>(nx, acc, As, Bs, srn, Qb, qlast, Re, rt, nr, ldp, rn, tid, w, h, c, hsc, rnext);
        if (ballot(self >= rt && self < rt + kTileRows)) {
            const int sr = self >= rt && self < rt + kTileRows ? (int)(self - rt) : -1;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    acc[b][v] = b * 32 + mfma_row(v, h) == sr ? -__builtin_inff() : acc[b][v];
        }
        if (ntiles <= 4 || rt == own * kTileRows) {
            // few references, or the queries' own tile: groups of four
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int v = 0; v < 16; v += 4)
                    top_insert(top, fmaxf(fmaxf(acc[b][v], acc[b][v + 1]), fmaxf(acc[b][v + 2], acc[b][v + 3])));
            continue;
        }
        float m[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            m[b] = acc[b][0];
#pragma unroll
            for (int v = 1; v < 16; ++v) m[b] = fmaxf(m[b], acc[b][v]);
        }
        if (ntiles <= 48) {   // groups of 16
#pragma unroll
            for (int b = 0; b < 4; ++b) top_insert(top, m[b]);
        } else {
            top_insert(top, fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3])));
        }
    }
    // the best 32 of both halves' groups, sorted descending
    float z[kListW];
#pragma unroll
    for (int q = 0; q < kListW; ++q) z[q] = fmaxf(top[q], xor_f32(top[kListW - 1 - q], 32));
#pragma unroll
    for (int j = kListW / 2; j > 0; j >>= 1)
#pragma unroll
        for (int q = 0; q < kListW; ++q)
            if ((q & j) == 0) {
                const float a = z[q], b = z[q + j];
                z[q] = fmaxf(a, b);
                z[q + j] = fminf(a, b);
            }
    if (qr < nq && h == 0) {
        f32x4* out = (f32x4*)(gtop + (qr * P + p) * kListW);
#pragma unroll
        for (int q = 0; q < kListW; q += 4) out[q / 4] = f32x4{z[q], z[q + 1], z[q + 2], z[q + 3]};
    }
}

// lims[row] = the kp-th best of the row's P lists of group scores, lowered by
// err (|q| + max|r|)^2 in scaled units.  Half a wave per row.  ecert > 0: rows
// are certified with the bound ecert (|q| + max|r|)^2; where that is not below
// the kp-th distance nothing can be, and the gate is +inf: the row goes to the
// exhaustive search without collecting candidates, all of which would pass (one
// row 10^6 times the others, 20,000 x 50: 4 of 22.8 ms).
__global__ __launch_bounds__(256) void gate_select_kernel(const float* __restrict__ gtop, int64_t nq, int P, int kp,
                                                          const float* __restrict__ qn,
                                                          const unsigned* __restrict__ rmax_bits,
                                                          const unsigned* __restrict__ qmax_bits, float err,
                                                          float ecert, float* __restrict__ lims)
{
    const int64_t row = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);
    const int lane = threadIdx.x & 63, c = lane & 31;
    if (row - (lane >> 5) >= nq) return;   // the whole wave
    const int64_t r = row < nq ? row : nq - 1;
    float a = gtop[r * P * kListW + c];
    for (int p = 1; p < P; ++p) {
        // two descending lists: the larger of entry i and entry 31 - i are
        // the best 32, a bitonic sequence
        a = fmaxf(a, gtop[(r * P + p) * kListW + (kListW - 1 - c)]);
#pragma unroll
        for (int j = 16; j > 0; j >>= 1) {
            const float o = xor_f32(a, j);
            a = (c & j) == 0 ? fmaxf(a, o) : fminf(a, o);
        }
    }
    if (c == kp - 1 && row < nq) {
        const float sc = qmax_bits ? query_scale(*qmax_bits, *rmax_bits) * split_scale(*rmax_bits) : 1.0f;
        const float nrm = sqrtf(qn[row]) + sqrtf(__uint_as_float(*rmax_bits));
        const bool hopeless = ecert > 0.0f && ecert * nrm * nrm >= qn[row] - 2.0f * a / sc;
        lims[row] = hopeless ? __builtin_inff() : a - err * nrm * nrm * sc;
    }
}

constexpr int kCandCap = 256;   // entries of a row's buffer

// Rows lr0 .. lr0 + 31 of one wave (counts n32, gates lim32 in LDS) whose
// buffers have no room for another tile's 128 keep their best 32 by (distance,
// index) and raise their gate to the kp-th of them.  self32 (nullable): the
// rows' own indices, which are dropped here (counted, one would take the place
// of the kp-th neighbour).
__device__ inline void compact_rows(uint64_t* buf, uint32_t rstride, uint32_t* n32, float* lim32,
                                    const int32_t* self32, int lr0, const float* qnb, int kp, float m2, float sc,
                                    float rmax)
{
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const uint32_t n = lane < 32 ? n32[lane] : 0u;
    for (uint64_t m = ballot(n > kCandCap - kTileRows); m; m &= m - 1) {
        const int r = __builtin_ctzll(m);
        const uint32_t nc = bcast_u32(n, r);
        const float sq = qnb[lr0 + r];
        const uint32_t self = self32 ? (uint32_t)self32[r] : 0xFFFFFFFFu;
        uint64_t* b = buf + (uint32_t)(lr0 + r) * rstride;
        auto key_of = [&](uint64_t x) { return make_key(fmaf(m2, __uint_as_float((uint32_t)(x >> 32)), sq), (uint32_t)x); };
        uint64_t best = kEmptyCand;
        for (uint32_t e = 0; e < nc; e += 64) {
            const uint64_t x = e + lane < nc ? b[e + lane] : ~0ull;
            const uint64_t key = e + lane < nc && (uint32_t)x != self ? key_of(x) : kEmptyCand;
            best = seg_merge_sorted<64>(best, seg_sort<64>(key));
        }
        const uint64_t last = bcast_u64(best, kListW - 1);
        const float t = key_d2(bcast_u64(best, kp - 1));
        // the entries up to the 32nd key move to the front
        uint32_t kept = 0;
        for (uint32_t e = 0; e < nc; e += 64) {
            const uint64_t x = e + lane < nc ? b[e + lane] : 0ull;
            const bool keep = e + lane < nc && (uint32_t)x != self && key_of(x) <= last;
            const uint64_t km = ballot(keep);
            if (keep) b[kept + rank_below(km)] = x;
            kept += (uint32_t)popc64(km);
        }
        if (lane == 0) {
            n32[r] = kept;
            lim32[r] = fmaxf(lim32[r], (0.5f * (sq - t) - 4.76837158e-07f * (sq + t + rmax)) * sc);   // 8u = 2^-21
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
}

// The gated pass: the tiles and pipeline of exact_tile_kernel; a score that
// reaches its row's gate is appended, as (score, index), to the row's buffer
// of kCandCap entries for this split (part[(row * S + s) * kCandCap ..], counts
// in LDS, then cnt[row * S + s]).  A row belongs to one wave, so appending
// needs no other wave.  When a buffer has no room for another tile's 128, its
// wave keeps the row's best 32 by (distance, index), its own index left out, and
// raises the gate to the kp-th of them (compact_rows): the keys the sorted
// lists of exact_tile_kernel would keep.  Rare where a row's neighbours are
// spread over the references; where they follow each other (rows sorted by
// cluster, position or time) the gate's groups are near-copies and several
// hundred references pass it.

template <int OUT, bool ARES>
__global__ __launch_bounds__(256, 2) void exact_append_kernel(
    const void* __restrict__ Qs, const float* __restrict__ qn, int64_t nq, const void* __restrict__ Rs,
    const float* __restrict__ rn, int64_t nr, int ldp, const int32_t* __restrict__ q_self, int self_mode,
    int64_t self_base, int kp, int64_t split_len, int S, const unsigned* __restrict__ rmax_bits,
    const unsigned* __restrict__ qmax_bits, const float* __restrict__ lims, uint64_t* part, uint32_t* __restrict__ cnt)
{
    using C = TileCfg<OUT>;
    using E = typename C::E;
    constexpr int LROW = C::LROW, AROW = ARES ? C::AROW : LROW;
    __shared__ __attribute__((aligned(16))) E As[kTileRows * AROW];
    __shared__ __attribute__((aligned(16))) E Bs[kTileRows * LROW];
    __shared__ float srn[kTileRows];
    __shared__ uint32_t scnt[kTileRows];
    __shared__ float slim[kTileRows];
    __shared__ int32_t sself[kTileRows];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, c = lane & 31;
    const int64_t q0 = (int64_t)blockIdx.x * kTileRows;
    const int s = blockIdx.y;
    const int64_t rbeg = (int64_t)s * split_len;
    const int64_t rend = rbeg + split_len < nr ? rbeg + split_len : nr;
    const float sc = qmax_bits ? query_scale(*qmax_bits, *rmax_bits) * split_scale(*rmax_bits) : 1.0f;
    const float rmax = __uint_as_float(*rmax_bits);
    const float m2 = -2.0f / sc, hsc = 0.5f * sc;
    if (tid < kTileRows) {
        scnt[tid] = 0u;
        slim[tid] = q0 + tid < nq ? lims[q0 + tid] : __builtin_inff();   // rows past nq take nothing
        const int64_t qr = q0 + tid;
        sself[tid] = qr >= nq ? -1 : (self_mode == 1 ? (int32_t)(self_base + qr) : (self_mode == 2 ? q_self[qr] : -1));
    }
    const E* Qb = (const E*)Qs + q0 * ldp;
    const E* Re = (const E*)Rs;
    const int qlast = nq - q0 > kTileRows ? kTileRows - 1 : (int)(nq - q0) - 1;
    if (ARES) load_queries<E, AROW>(As, Qb, qlast, ldp, tid);
    StepRegs nx;
    load_step<E, ARES>(nx, Qb, qlast, Re, rbeg, rend, 0, ldp, rn, tid);
    __syncthreads();
    float lim[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) lim[v] = slim[w * 32 + mfma_row(v, h)];
    uint64_t* buf = part + (q0 * S + s) * kCandCap;   // row lr at buf + lr * S * kCandCap
    const uint32_t rstride = (uint32_t)S * kCandCap;
    for (int64_t rt = rbeg; rt < rend; rt += kTileRows) {
        f32x16 acc[4];
        tile_gemm<OUT, ARES, kByColumn>(nx, acc, As, Bs, srn, Qb, qlast, Re, rt, rend, ldp, rn, tid, w, h, c, hsc);
        bool full = false;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            uint64_t any = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) any |= ballot(acc[blk][v] >= lim[v]);
            if (!any) continue;
            const uint32_t j = (uint32_t)rt + blk * 32 + c;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                // columns past the references score -inf, which a gate of -inf
                // (fewer groups than kp) lets pass: not references
                if (acc[blk][v] >= lim[v] && j < (uint32_t)rend) {
                    const int lr = w * 32 + mfma_row(v, h);
                    const uint32_t pos = atomicAdd(&scnt[lr], 1u);   // below kCandCap: see `full`
                    buf[(uint32_t)lr * rstride + pos] = ((uint64_t)__float_as_uint(acc[blk][v]) << 32) | j;
                    full = full || pos >= kCandCap - kTileRows;
                }
            }
        }
        if (ballot(full)) {
            compact_rows(buf, rstride, scnt + w * 32, slim + w * 32, sself + w * 32, w * 32, qn + q0, kp, m2, sc, rmax);
#pragma unroll
            for (int v = 0; v < 16; ++v) lim[v] = slim[w * 32 + mfma_row(v, h)];
        }
    }
    __syncthreads();
    if (tid < kTileRows && q0 + tid < nq) cnt[(q0 + tid) * S + s] = scnt[tid];
}

// ------------------------------------------------------------ rank counts

constexpr int kRankP = 16;   // probes per query row (the quality metrics' k <= 16)
constexpr int kRankFlush = 1024;   // queued pairs that are worth a recheck pass
constexpr int kRankQueue = kTileRows * kTileRows + kRankFlush;

// Squared norms from 2^124 on: sums and distances may overflow FP32, and bound
// nothing.
__device__ inline bool rank_wide(unsigned mx) { return mx >= (127u + 124u) << 23; }

// The counts of rank_tile_kernel below where rank_wide, every pair decided by
// its canonical distance; nothing is done otherwise.  A workgroup takes a query,
// a 16-lane group a reference.  (In the tile pass itself this branch cost
// 3.6% of a 70,000 x 784 call.)
__global__ __launch_bounds__(256) void rank_wide_kernel(const float* __restrict__ Zf, int64_t ldf, int d, int64_t q0,
                                                        int64_t nq, int64_t n, const uint64_t* __restrict__ probes,
                                                        const unsigned* __restrict__ rmax_bits,
                                                        uint32_t* __restrict__ counts)
{
    if (!rank_wide(*rmax_bits)) return;
    const int g = threadIdx.x & 15;
    for (int64_t q = blockIdx.x; q < nq; q += gridDim.x) {
        const uint64_t key = probes[q * kRankP + g];
        uint32_t num = 0;
        for (int64_t r0 = 0; r0 < n; r0 += 16) {
            const int64_t r = r0 + (threadIdx.x >> 4);
            const bool act = r < n && r != q0 + q;
            const float d2 = dist_g16<KNN_F32>(Zf, (q0 + q) * ldf, Zf, (act ? r : 0) * ldf, d, act);
            num += act && key != kEmptyCand && make_key(d2, (uint32_t)r) < key ? 1u : 0u;
        }
        if (num) atomicAdd(&counts[q * kRankP + g], num);
    }
}

// For every query row q and each of its probes (keys (canonical d2, index),
// ascending; kEmptyCand pads), counts[q][p] = the number of reference rows
// m != self(q) whose key (canonical FP32 d2(q, m), m) is below the probe's
// key: the probe's rank minus one.  The tiles and pipeline of the exact
// search on split rows, operands swapped (a lane's sums belong to one query:
// its probes, as scores, and its counts sit in registers), S reference splits
// whose counts are added into counts, zeroed beforehand.  A score further from
// a probe's than the slack (the GEMM bound with the tile's largest norm, the
// parts' absolute error, plus the canonical distance's) decides it; what is left is queued (the pair and
// its range of undecided probes) in the workgroup's global queue, which is
// worked off once it holds 1,024 pairs: 16-lane groups form the pairs'
// canonical FP32 distances from the rows Zf, four pairs in flight, in the order
// dist_g16 sums, and count them exactly.  No pair is decided any other way.
// With LISTS the pass also appends, as exact_append_kernel does, what reaches
// the row's gate, for X's exact k-NN.
// What bounds it: the three products per element, then rechecks (two rows of
// 4 d bytes each), whose number is proportional to the slack; forming the sums
// in segments makes the bound 208 u |q||r| where one chain of FP32 additions had
// 1,572 (d = 784), some 38 rechecks per tile instead of 250.  70,000 x 784, k =
// 10: 104 ms with FP32 MFMA, a histogram in LDS and every tile's rows streamed
// again for its rechecks; 44 ms now.
template <bool LISTS, bool ARES, int NP>
__global__ __launch_bounds__(256, 2) void rank_tile_kernel(
    const _Float16* __restrict__ Qs, const float* __restrict__ qn, int64_t nq, const _Float16* __restrict__ Rs,
    const float* __restrict__ rn, int64_t nr, int lds, const float* __restrict__ Qf, const float* __restrict__ Zf,
    int64_t ldf, int d, int64_t self_base, const uint64_t* __restrict__ probes, const unsigned* __restrict__ rmax_bits,
    float ec_dot, float ec_norm, float edir, float eabs, float eden, int S, int64_t split_len, uint32_t* __restrict__ counts,
    uint64_t* gqueue, int kp, const float* __restrict__ lims, uint64_t* part, uint32_t* __restrict__ cnt)
{
    using C = TileCfg<KNN_SPLIT>;
    using E = typename C::E;
    constexpr int LROW = C::LROW, AROW = ARES ? C::AROW : LROW;
    __shared__ __attribute__((aligned(16))) E As[kTileRows * AROW];
    __shared__ __attribute__((aligned(16))) E Bs[kTileRows * LROW];
    __shared__ __attribute__((aligned(16))) float srn[kTileRows];
    __shared__ uint64_t skey[kTileRows * NP];
    __shared__ uint32_t sadd[kTileRows * NP];   // the rechecks' counts
    __shared__ uint32_t scnt[kTileRows];
    __shared__ float slim[kTileRows];
    __shared__ uint32_t qcount;
    uint64_t* queue = gqueue + (int64_t)blockIdx.x * kRankQueue;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, c = lane & 31;
    // workgroup = (query block, reference split): splits rbeg .. rend
    const int64_t q0 = (int64_t)(blockIdx.x / S) * kTileRows;
    const int sp = blockIdx.x % S;
    const int64_t rbeg = (int64_t)sp * split_len;
    const int64_t rend = rbeg + split_len < nr ? rbeg + split_len : nr;
    if (rank_wide(*rmax_bits)) {
        // rank_wide_kernel's: empty lists, whose rows are searched exhaustively
        if (LISTS && tid < kTileRows && q0 + tid < nq) cnt[(q0 + tid) * S + sp] = 0u;
        return;
    }
    const float scale = split_scale(*rmax_bits), sc = scale * scale, hsc = 0.5f * sc, m2 = -2.0f / sc;
    for (int e = tid; e < kTileRows * NP; e += 256) {
        const int64_t qr = q0 + e / NP;
        skey[e] = qr < nq ? probes[qr * kRankP + e % NP] : kEmptyCand;
        sadd[e] = 0u;
    }
    if (tid < kTileRows) {
        scnt[tid] = 0u;
        // a gate of -inf (fewer groups than kp) would let the columns past the
        // references pass, whose scores are -inf
        slim[tid] = LISTS && q0 + tid < nq ? fmaxf(lims[q0 + tid], -3.402823466e38f) : __builtin_inff();
    }
    if (tid == 0) qcount = 0u;
    const E* Qb = (const E*)Qs + q0 * lds;
    const E* Re = (const E*)Rs;
    const int qlast = nq - q0 > kTileRows ? kTileRows - 1 : (int)(nq - q0) - 1;
    if (ARES) load_queries<E, AROW>(As, Qb, qlast, lds, tid);
    StepRegs nx;
    load_step<E, ARES>(nx, Qb, qlast, Re, rbeg, rend, 0, lds, rn, tid);
    __syncthreads();
    // this lane's query: its probes as scores (+inf: none), counts and gate
    const int lq = w * 32 + c;
    const int64_t qr = q0 + lq;
    const float sq = qr < nq ? qn[qr] : 0.0f, qa = sqrtf(sq);
    const int64_t self = qr < nq ? self_base + qr : -1;
    float ts[NP], lim = slim[lq], mx = 0.0f, tlow = __builtin_inff();
    uint32_t num[NP];
    int nv = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint64_t key = skey[lq * NP + p];
        const bool on = key != kEmptyCand;
        ts[p] = on ? 0.5f * (sq - key_d2(key)) * sc : __builtin_inff();
        tlow = on ? ts[p] : tlow;   // the farthest probe's
        mx = on ? key_d2(key) : mx;
        nv += on ? 1 : 0;
        num[p] = 0u;
    }
    // the slack, in score units, with a tile's largest norm |r|^2: hsc (e2 + 2 edir
    // (mx + e2)) + eabs scale (|q| + |r|) + eden with e2 = ec_dot |q||r| + ec_norm
    // (|q|^2 + |r|^2 + mx), as slr |r| + slt |r|^2 + sl0
    const float hx = hsc * (1.0f + 2.0f * edir), slr = hx * ec_dot * qa + eabs * scale, slt = hx * ec_norm;
    const float sl0 = hx * ec_norm * (sq + mx) + 2.0f * hsc * edir * mx + eabs * scale * qa + eden;
    uint64_t* buf = LISTS ? part + (q0 * S + sp) * kCandCap : nullptr;
    const uint32_t rstride = (uint32_t)S * kCandCap;
    for (int64_t rt = rbeg; rt < rend; rt += kTileRows) {
        f32x16 acc[4];
        tile_gemm<KNN_SPLIT, ARES, kSegmented>(nx, acc, As, Bs, srn, Qb, qlast, Re, rt, rend, lds, rn, tid, w, h, c, hsc);
        // the tile's largest norm (rows past rend: +inf, left out)
        float tn = 0.0f;
        {
            const float a = srn[lane], b = srn[64 + lane];
            tn = fmaxf(a < __builtin_inff() ? a : 0.0f, b < __builtin_inff() ? b : 0.0f);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) tn = fmaxf(tn, xor_f32(tn, o));
        }
        const float sl = fmaf(slr, sqrtf(tn), fmaf(slt, tn, sl0));
        const bool diag = ballot(self >= rt && self < rt + kTileRows) != 0ull;
        const int sr = self >= rt && self < rt + kTileRows ? (int)(self - rt) : -1;
        bool full = false;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            float mxs = -__builtin_inff();
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const f32x4 x = *(const f32x4*)&srn[blk * 32 + 8 * v4 + 4 * h];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = 4 * v4 + e;
                    acc[blk][v] -= hsc * x[e];
                    if (diag) acc[blk][v] = blk * 32 + mfma_row(v, h) == sr ? -__builtin_inff() : acc[blk][v];
                    mxs = fmaxf(mxs, acc[blk][v]);
                }
            }
            // nothing near any probe or the gate
            if (!ballot(mxs + sl >= tlow || (LISTS && mxs >= lim))) continue;
            // rolled, the score picked by index: 16 copies of the body spilled
            // hundreds of registers and outgrew the instruction cache
            const f32x16 cur = acc[blk];
#pragma unroll 1
            for (int v = 0; v < 16; ++v) {
                const float x = cur[v], xm = x - sl, xp = x + sl;
                bool und = false;
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const bool below = xm > ts[p], poss = xp >= ts[p];
                    num[p] += below ? 1u : 0u;
                    und = und || (below != poss);
                }
                const uint32_t j = (uint32_t)rt + blk * 32 + mfma_row(v, h);
                if (und) {
                    int a = 0, b = 0;
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        a += xp >= ts[p] ? 1 : 0;
                        b += xm > ts[p] ? 1 : 0;
                    }
                    // probes nv - a .. nv - b - 1 are undecided
                    const uint32_t slot = atomicAdd(&qcount, 1u);
                    queue[slot] = ((uint64_t)j << 32) | (uint32_t)(lq << 10 | (nv - a) << 5 | (nv - b));
                }
                if (LISTS && x >= lim) {
                    const uint32_t pos = atomicAdd(&scnt[lq], 1u);
                    buf[(uint32_t)lq * rstride + pos] = ((uint64_t)__float_as_uint(x) << 32) | j;
                    full = full || pos >= kCandCap - kTileRows;
                }
            }
        }
        if (LISTS && ballot(full)) {
            // a row's own score is -inf: never among the best
            compact_rows(buf, rstride, scnt + w * 32, slim + w * 32, nullptr, w * 32, qn + q0, kp, m2, sc,
                         __uint_as_float(*rmax_bits));
            lim = slim[lq];
        }
        __syncthreads();   // the queue is complete
        const int nqd = (int)qcount;
        if (nqd >= kRankFlush || (rt + kTileRows >= rend && nqd > 0)) {
            // group tid / 16 takes pairs base + tid / 16 + 16 m; one past the
            // end repeats the last and drops the sum
            const int g = tid & 15;
            for (int base = 0; base < nqd; base += 64) {
                uint64_t ent[4];
                const float *a[4], *b[4];
                float sum[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int e = base + (tid >> 4) + 16 * m;
                    ent[m] = queue[e < nqd ? e : nqd - 1];
                    a[m] = Qf + (q0 + (int64_t)((uint32_t)ent[m] >> 10)) * ldf;
                    b[m] = Zf + (int64_t)(ent[m] >> 32) * ldf;
                    sum[m] = 0.0f;
                }
#pragma unroll 2
                for (int t = g; t < d; t += 16) {
                    float x[4], y[4];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        x[m] = a[m][t];
                        y[m] = b[m][t];
                    }
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const float df = x[m] - y[m];
                        sum[m] = fmaf(df, df, sum[m]);
                    }
                }
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const float dc = wave_sum16(sum[m]);
                    const int e = base + (tid >> 4) + 16 * m;
                    if (e < nqd && g < NP) {
                        // lane g: probe g, if it is one of the undecided
                        const uint32_t lo = (uint32_t)ent[m];
                        const int lr = (int)(lo >> 10), p1 = (int)((lo >> 5) & 31u), p0 = (int)(lo & 31u);
                        if (g >= p1 && g < p0 && make_key(dc, (uint32_t)(ent[m] >> 32)) < skey[lr * NP + g])
                            atomicAdd(&sadd[lr * NP + g], 1u);
                    }
                }
            }
            __syncthreads();   // the queue is read
            if (tid == 0) qcount = 0u;
        }
        // (the next tile's first barrier orders the reset before its appends)
    }
    __syncthreads();
    if (qr < nq) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t other = xor_u32(num[p], 32);   // the other half's references
            if (h == 0 && p < nv) atomicAdd(&counts[qr * kRankP + p], num[p] + other + sadd[lq * NP + p]);
        }
    }
    if (LISTS && tid < kTileRows && q0 + tid < nq) cnt[(q0 + tid) * S + sp] = scnt[tid];
}

// The same counts for a low-dimensional space (d <= kRankDirectD, e.g. a 2-D
// embedding), by direct canonical FP32 distances: there the norm
// expansion's error bound is wider than neighbour distances, so a GEMM pass
// would recheck nearly every pair.  Thread = query row; its probe keys and
// counts sit in registers; the reference rows of the workgroup's split
// stream through LDS in tiles of 256, and the splits' counts are added into
// counts (zeroed beforehand).  Exact in the canonical precision, no
// ambiguity.  A reference below a probe's key (distance, index) is one whose
// distance bits are below the probe's, or equal to them with a smaller index:
// before the probe's own position "below bits + 1", behind it "below bits".  So
// the groups of 8 references that hold no probe and not the query, all but a few
// for a wave, take one 32-bit comparison and an add per probe.  Bound by those
// (70,000 x 2, 10 probes: 4.22 ms; 5.65 with 64-bit keys for 16 probes).
constexpr int kRankDirectD = 16;
// Workgroups per rank_tile_kernel launch: each holds a 136 KiB queue of
// undecided pairs (272 MiB per launch) and, with lists, 256 KiB of buffers.
constexpr int64_t kRankBlocks = 2048;
constexpr int kRankMaxSplits = 8;   // reference splits of the rank pass

// DC = d when it is a compile-time constant (2, 3), 0 for any d <= 16; NP: probes
// held (at most as many are used).
template <int DC, int NP>
__global__ __launch_bounds__(256) void rank_direct_kernel(const float* __restrict__ Xs, int64_t n, int ldp, int dd,
                                                          const uint64_t* __restrict__ probes, int64_t split_len,
                                                          uint32_t* __restrict__ counts)
{
    const int d = DC ? DC : dd;
    constexpr int DT = DC ? DC : kRankDirectD;   // coordinates held per row
    __shared__ float tile[256][DT + 1];
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t rbeg = (int64_t)blockIdx.y * split_len, rend = rbeg + split_len < n ? rbeg + split_len : n;
    const bool live = q < n;
    float xq[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) xq[t] = live && t < d ? Xs[q * ldp + t] : 0.0f;
    // a probe that is not used counts what it may
    uint32_t pd[NP], pi[NP], cnt[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint64_t key = live ? probes[q * kRankP + p] : 0ull;
        pd[p] = (uint32_t)(key >> 32);
        pi[p] = key_idx(key);
        cnt[p] = 0u;
    }
    for (int64_t r0 = rbeg; r0 < rend; r0 += 256) {
        __syncthreads();
        {
            const int64_t r = r0 + threadIdx.x;
#pragma unroll
            for (int t = 0; t < DT; ++t) tile[threadIdx.x][t] = r < rend && t < d ? Xs[r * ldp + t] : 0.0f;
        }
        __syncthreads();
        const int nr = (int)(rend - r0 < 256 ? rend - r0 : 256);
        // bounds before the probes' positions, and the wave's groups of 8 with a
        // probe or a query
        uint32_t below[NP];
        const uint32_t own = (uint32_t)q - (uint32_t)r0;
        uint32_t mask = own < 256u ? 1u << (own >> 3) : 0u;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t o = pi[p] - (uint32_t)r0;
            below[p] = pd[p] + ((int32_t)o >= 0 ? 1u : 0u);
            mask |= o < 256u ? 1u << (o >> 3) : 0u;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mask |= xor_u32(mask, o);
        mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)mask);
        for (int j0 = 0; j0 < nr; j0 += 8) {
            uint32_t b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                b[u] = __float_as_uint(fmaxf(direct_d2<DT>(xq, tile[j0 + u < nr ? j0 + u : j0], d), 0.0f));
            if (j0 + 8 <= nr && !((mask >> (j0 >> 3)) & 1u)) {
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int p = 0; p < NP; ++p) cnt[p] += b[u] < below[p] ? 1u : 0u;
                continue;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t m = (uint32_t)r0 + j0 + u;
                if (j0 + u < nr && m != (uint32_t)q) {
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        cnt[p] += b[u] < pd[p] || (b[u] == pd[p] && m < pi[p]) ? 1u : 0u;
                }
            }
            // behind this group for its probes
#pragma unroll
            for (int p = 0; p < NP; ++p) below[p] -= (pi[p] - (uint32_t)r0) >> 3 == (uint32_t)(j0 >> 3) ? 1u : 0u;
        }
    }
    if (live) {
#pragma unroll
        for (int p = 0; p < NP; ++p) atomicAdd(&counts[q * kRankP + p], cnt[p]);   // the splits' counts add up
    }
}

// Exact k-NN in a low-dimensional space (d <= kRankDirectD, e.g. a 2-D
// embedding): there the norm expansion's error bound exceeds neighbour
// distances, so GEMM certificates fail; instead every pair's canonical FP32
// distance is formed directly (thread = query row, reference rows through
// LDS, the canonical sum as in rank_direct_kernel) and each thread keeps
// its KM smallest keys (canonical d2, index) in registers.  Workgroup
// (query block, reference split) writes its sorted list, padded to kListW,
// in the split-list layout merge_rerank_kernel merges.
template <int DT, int DC, int KM>
__global__ __launch_bounds__(256) void exact_direct_kernel(
    const void* __restrict__ Q, int64_t ldq, int64_t nq, const void* __restrict__ R, int64_t ldr, int64_t nr,
    int dd, const int32_t* __restrict__ q_self, int self_mode, int64_t self_base, int k, int64_t split_len, int S,
    uint64_t* __restrict__ part)
{
    const int d = DC ? DC : dd;
    constexpr int DT_ = DC ? DC : kRankDirectD;
    __shared__ float tile[256][DT_ + 1];
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = blockIdx.y;
    const int64_t rbeg = (int64_t)s * split_len, rend = rbeg + split_len < nr ? rbeg + split_len : nr;
    const bool live = q < nq;
    const int64_t self = !live ? -1 : (self_mode == 1 ? self_base + q : (self_mode == 2 ? (int64_t)q_self[q] : -1));
    float xq[DT_];
#pragma unroll
    for (int t = 0; t < DT_; ++t) xq[t] = live && t < d ? elem<DT>::ld(Q, q * ldq + t) : 0.0f;
    uint64_t list[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) list[j] = kEmptyList;
    uint64_t kth = kEmptyList;   // list[k - 1]
    for (int64_t r0 = rbeg; r0 < rend; r0 += 256) {
        __syncthreads();
        {
            const int64_t r = r0 + threadIdx.x;
#pragma unroll
            for (int t = 0; t < DT_; ++t) tile[threadIdx.x][t] = r < rend && t < d ? elem<DT>::ld(R, r * ldr + t) : 0.0f;
        }
        __syncthreads();
        const int nt = (int)(rend - r0 < 256 ? rend - r0 : 256);
        // 32 references at a time: first the gate against the list's k-th key
        // as it stood (a bit per passing reference), then the passing ones
        // inserted in index order, each re-tested against the current k-th
        // key, so a wave runs as many insertion steps as its busiest lane
        for (int j0 = 0; j0 < nt; j0 += 32) {
            const int jn = nt - j0 < 32 ? nt - j0 : 32;
            uint32_t mask = 0u;
            for (int jj = 0; jj < jn; ++jj) {
                const int64_t m = r0 + j0 + jj;
                const uint64_t key = make_key(direct_d2<DT_>(xq, tile[j0 + jj], d), (uint32_t)m);
                mask |= (key < kth && m != self) ? 1u << jj : 0u;
            }
            while (mask) {
                const int jj = __builtin_ctz(mask);
                mask &= mask - 1u;
                const uint64_t key = make_key(direct_d2<DT_>(xq, tile[j0 + jj], d), (uint32_t)(r0 + j0 + jj));
                if (key < kth) {
                    // insertion into the ascending list; entries past k stay empty
#pragma unroll
                    for (int j = KM - 1; j >= 1; --j) {
                        const uint64_t a = list[j - 1], b = list[j];
                        list[j] = j < k ? (key < a ? a : (key < b ? key : b)) : b;
                    }
                    list[0] = key < list[0] ? key : list[0];
#pragma unroll
                    for (int j = 0; j < KM; ++j) kth = j == k - 1 ? list[j] : kth;
                }
            }
        }
    }
    if (live) {
        uint64_t* out = part + (q * S + s) * kListW;
#pragma unroll
        for (int c = 0; c < kListW; ++c) out[c] = c < KM ? list[c] : kEmptyList;
    }
}

// Small searches in FP32: every pair's canonical distance, one launch, no
// staging, no scratch.  A wave owns a query (WQ = 4: four waves, a quarter of
// the references each, their lists merged at the end); 64 references at a time pass
// through LDS, 32 coordinates each, lane = reference, its distance summed in
// the 16 partial sums and the tree of dist_g16.  Keys below the list's k-th
// enter the wave's 64-entry sorted list, a few one by one, more by a sort and a
// merge.  The next chunk is loaded while this one is summed.  500 x 50 (k =
// 15): 23 us of kernel, 42 of call, against 85 and 107 of the staged route (72 us
// filling lists from one tile per workgroup).
constexpr int64_t kSmallRefs = 4096;
constexpr double kSmallWork = 3e9;   // queries * references * (6 d + 150) instructions

template <int DT, int WQ>
__global__ __launch_bounds__(256) void exact_small_kernel(
    const void* __restrict__ Q, int64_t ldq, int nq, const void* __restrict__ R, int64_t ldr, int nr, int d,
    const int32_t* __restrict__ q_self, int self_mode, int k, int out_kind, int32_t* __restrict__ out_idx,
    float* __restrict__ out_dist)
{
    constexpr int CW = 32;         // coordinates per chunk
    constexpr int TR = 64 * WQ;    // references per tile
    __shared__ __attribute__((aligned(16))) float rs[TR][CW + 1];
    __shared__ __attribute__((aligned(16))) float qs[4][CW];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int q0 = blockIdx.x * (4 / WQ), q = WQ == 4 ? q0 : q0 + w;
    const int row = WQ == 4 ? tid : lane, qw = WQ == 4 ? 0 : w;   // this lane's row of the tile, its query's of qs
    const int qc = q < nq ? q : nq - 1;
    const int self = self_mode == 1 ? qc : (self_mode == 2 ? q_self[qc] : -1);
    const int cc = tid & 31, rr = tid >> 5;   // staging: column cc of rows rr, rr + 8, ...
    const int qr = q0 + (rr & 3) < nq ? q0 + (rr & 3) : nq - 1;
    float xr[8 * WQ], xq;
    auto fetch = [&](int base, int c0) {
        const int t = c0 + cc;
#pragma unroll
        for (int u = 0; u < 8 * WQ; ++u) {
            const int r = base + rr + 8 * u;
            xr[u] = t < d ? elem<DT>::ld(R, (int64_t)(r < nr ? r : nr - 1) * ldr + t) : 0.0f;
        }
        xq = t < d ? elem<DT>::ld(Q, (int64_t)qr * ldq + t) : 0.0f;
    };
    uint64_t list = kEmptyList;
    fetch(0, 0);
    for (int base = 0; base < nr; base += TR) {
        float s[16];
#pragma unroll
        for (int g = 0; g < 16; ++g) s[g] = 0.0f;
        for (int c0 = 0; c0 < d; c0 += CW) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8 * WQ; ++u) rs[rr + 8 * u][cc] = xr[u];
            if (rr < 4) qs[rr][cc] = xq;
            __syncthreads();
            if (c0 + CW < d) fetch(base, c0 + CW);
            else if (base + TR < nr) fetch(base + TR, 0);
            // coordinates past d are zero on both sides: the sums keep their bits
#pragma unroll
            for (int t = 0; t < CW; t += 4) {
                const f32x4 x = *(const f32x4*)&qs[qw][t];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float df = x[e] - rs[row][t + e];
                    s[(t + e) & 15] = fmaf(df, df, s[(t + e) & 15]);
                }
            }
        }
#pragma unroll
        for (int j = 8; j > 0; j >>= 1)
#pragma unroll
            for (int g = 0; g < j; ++g) s[g] = s[g] + s[g + j];
        const int j = base + row;
        const uint64_t key = j < nr && j != self ? make_key(s[0], (uint32_t)j) : kEmptyCand;
        uint64_t m = ballot(key < bcast_u64(list, k - 1));
        if (popc64(m) > 6) {
            list = seg_merge_sorted<64>(list, seg_sort<64>(key));
        } else {
            for (; m; m &= m - 1) {
                // entries above the key move up one place, the first takes it
                const uint64_t x = bcast_u64(key, __builtin_ctzll(m)), up = shift_up_u64(list);
                list = umin64(list, umax64(up, x));
            }
        }
    }
    if constexpr (WQ == 4) {
        // the four waves' lists
        uint64_t* all = (uint64_t*)&rs[0][0];
        __syncthreads();
        all[tid] = list;
        __syncthreads();
        if (w != 0) return;
        list = seg_merge_sorted<64>(seg_merge_sorted<64>(list, all[64 + lane]),
                                    seg_merge_sorted<64>(all[128 + lane], all[192 + lane]));
    }
    if (q < nq && lane < k) {
        const float d2 = key_d2(list);
        out_idx[(int64_t)q * k + lane] = (int32_t)key_idx(list);
        out_dist[(int64_t)q * k + lane] = out_kind == KNN_OUT_L2 ? sqrtf(d2) : d2;
    }
}

// ------------------------------------------------------------ merge/rerank

// One wave per query row.  Merges the S split lists (S x 32 keys), keeps
// the best kp by GEMM distance, re-ranks them with the canonical FP32
// direct-difference distance on the original inputs and writes the best k.
// With cnt (nullable) the splits hold cnt[row * S + s] unsorted (score, index)
// pairs of the gated pass instead, kCandCap apart, among them the row's own
// index; a score becomes the distance |q|^2 - 2 s / scale.
template <int DT>
__global__ __launch_bounds__(256) void merge_rerank_kernel(
    const uint64_t* __restrict__ part, const uint32_t* __restrict__ cnt, const int32_t* __restrict__ q_self,
    int self_mode, int64_t self_base, const unsigned* __restrict__ qmax_bits, int S, int64_t nq, int kp, int k,
    const void* __restrict__ Q, int64_t ldq, const void* __restrict__ R, int64_t ldr, int d,
    const float* __restrict__ qn, const unsigned* __restrict__ rmax_bits, float err_coef,
    float edir, float eabs, int certify, int64_t avail, int out_kind, int32_t* __restrict__ out_idx,
    float* __restrict__ out_dist, int32_t* __restrict__ fb_rows, int* __restrict__ fb_count)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= nq) return;
    // split lists (each sorted, 32 keys): even splits merge in lanes 0..31,
    // odd ones in lanes 32..63, keeping each half's 32 smallest; the two
    // halves then form one ascending 64-key sequence
    uint64_t k0;
    if (cnt) {
        const float sc = qmax_bits ? query_scale(*qmax_bits, *rmax_bits) * split_scale(*rmax_bits) : 1.0f;
        const float m2 = -2.0f / sc, sq = qn[row];
        const int64_t self = self_mode == 1 ? self_base + row : (self_mode == 2 ? (int64_t)q_self[row] : -1);
        k0 = kEmptyCand;
        for (int s = 0; s < S; ++s) {
            const uint32_t n = cnt[row * S + s];
            const uint64_t* b = part + (row * S + s) * kCandCap;
            for (uint32_t e = 0; e < n; e += 64) {
                const uint64_t x = e + lane < n ? b[e + lane] : 0ull;
                uint64_t key = make_key(fmaf(m2, __uint_as_float((uint32_t)(x >> 32)), sq), (uint32_t)x);
                if (e + lane >= n || (int64_t)(uint32_t)x == self) key = kEmptyCand;
                // nothing below the 32nd so far: skip the sort
                if (ballot(key < bcast_u64(k0, kListW - 1))) k0 = seg_merge_sorted<64>(k0, seg_sort<64>(key));
            }
        }
    } else {
        const int sp = lane >> 5;
        uint64_t acc = sp < S ? part[(row * S + sp) * kListW + (lane & 31)] : kEmptyCand;
        for (int b = 2; b < S; b += 2) {
            const uint64_t nk = b + sp < S ? part[(row * S + b + sp) * kListW + (lane & 31)] : kEmptyCand;
            acc = seg_merge_sorted<32>(acc, nk);
        }
        const uint64_t rv = shfl_xor_u64(acc, 31);
        k0 = seg_bitonic_merge<64>(sp ? rv : acc);
    }
    const uint64_t ck = lane < kp ? k0 : kEmptyCand;
    const bool cvalid = lane < kp && key_valid(ck);
    const int nvalid = popc64(ballot(cvalid));
    const float T = key_d2(bcast_u64(k0, kp - 1));
    const uint32_t myidx = key_idx(ck);

    float dd = 0.0f;
    for (int base = 0; base < kp; base += 4) {
        const int ci = base + (lane >> 4);
        const uint32_t cj = shfl_u32(myidx, ci < 64 ? ci : 0);
        const bool act = ci < kp && cj != 0xFFFFFFFFu;
        const float v = dist_g16<DT>(Q, row * ldq, R, (int64_t)cj * ldr, d, act);
        const float got = shfl_f32(v, ((lane - base) & 3) * 16);
        if (lane >= base && lane < base + 4) dd = got;
    }
    uint64_t nk = cvalid ? make_key(dd, myidx) : kEmptyCand;
    nk = seg_sort<64>(nk);
    if (lane < k) {
        const float d2 = key_d2(nk);
        out_idx[row * k + lane] = (int32_t)key_idx(nk);
        out_dist[row * k + lane] = out_kind == KNN_OUT_L2 ? sqrtf(d2) : d2;
    }
    if (certify) {
        const float Dk = key_d2(bcast_u64(nk, k - 1));
        const float qa = sqrtf(qn[row]);
        const float ra = sqrtf(__uint_as_float(*rmax_bits));
        // the absolute error of the queries' parts (2^-25 of a scaled unit,
        // taken twice), which (|q| + max|r|)^2 holds only where their norms are
        // not far above the references'
        const float E = err_coef * (qa + ra) * (qa + ra) + eabs * ra / query_scale(*qmax_bits, *rmax_bits);
        // fewer than kp keys: certain when there are no more candidates
        const bool cert = nvalid < kp ? (int64_t)nvalid >= avail : (Dk * (1.0f + edir) <= T - E && split_range(*rmax_bits) && !split_far(qn[row], *rmax_bits));
        if (!cert && lane == 0) {
            int p = atomicAdd(fb_count, 1);
            fb_rows[p] = (int32_t)row;
        }
    }
}

// --------------------------------------------------------------- fallback

// Exhaustive direct-difference k-NN for the rows listed in fb_rows.  The
// work is one canonical distance per (listed row, reference): reading the
// references bounds it, so how many workgroups share a row decides the time.
// The count is known only here: with cnt rows, each row's references are cut
// into P parts so that cnt * P workgroups run (P = 1 when the rows alone fill
// the grid); a part is at least the 256 references of one batch.  With P > 1
// every part's 32 best keys go to `lists` (room for `slots` lists; the split
// lists, already merged, are reused) and the workgroup that finishes last
// (counted in *done, zeroed beforehand) merges each row's parts.  One
// workgroup per row, whatever their count, had left one uncertified row of
// the 70,000 x 784 pixel set to a single workgroup: 64 ms of a 179 ms quality
// call, which now takes 116 ms, as without such a row.
// A wave takes 64 references per batch, four per 16-lane group in flight.
template <int DT>
__global__ __launch_bounds__(256) void exact_fallback_kernel(
    const int32_t* __restrict__ fb_rows, const int* __restrict__ fb_count,
    const void* __restrict__ Q, int64_t ldq, const void* __restrict__ R, int64_t ldr, int64_t nr,
    int d, const int32_t* __restrict__ q_self, int self_mode, int64_t self_base, int k, int out_kind,
    int32_t* __restrict__ out_idx, float* __restrict__ out_dist, uint64_t* lists, int64_t slots,
    unsigned* __restrict__ done)
{
    __shared__ uint64_t sl[4][64];
    __shared__ unsigned order_;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane & 15;
    const int cnt = *fb_count;
    if (cnt == 0) return;
    int64_t P = (slots < (int64_t)gridDim.x ? slots : (int64_t)gridDim.x) / cnt;
    const int64_t batches = ceil_div(nr, 256);
    P = P > batches ? batches : (P < 1 ? 1 : P);
    const int64_t jobs = (int64_t)cnt * P, per = ceil_div(batches, P) * 256;
    auto write_row = [&](int64_t row, uint64_t key) {
        if (lane < k) {
            const float d2 = key_d2(key);
            out_idx[row * k + lane] = (int32_t)key_idx(key);
            out_dist[row * k + lane] = out_kind == KNN_OUT_L2 ? sqrtf(d2) : d2;
        }
    };
    for (int64_t job = blockIdx.x; job < jobs; job += gridDim.x) {
        const int64_t row = fb_rows[job / P], c = job % P;
        const int64_t self = self_mode == 1 ? self_base + row : (self_mode == 2 ? (int64_t)q_self[row] : -1);
        const int64_t rbeg = c * per, rend = rbeg + per < nr ? rbeg + per : nr;
        uint64_t list = kEmptyList;
        for (int64_t base = rbeg + wv * 64; base < rend; base += 256) {
            uint64_t cand = kEmptyCand;
            for (int p0 = 0; p0 < 16; p0 += 4) {
                // pass p0 + u: references base + 4 (p0 + u) + group; their
                // loads of a coordinate step are issued together, each sum
                // in the order dist_g16 forms it
                float s[4];
                int64_t off[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t j = base + (p0 + u) * 4 + (lane >> 4);
                    off[u] = (j < rend ? j : rend - 1) * ldr;
                    s[u] = 0.0f;
                }
                for (int t = g; t < d; t += 16) {
                    const float xq = elem<DT>::ld(Q, row * ldq + t);
                    float xr[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) xr[u] = elem<DT>::ld(R, off[u] + t);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float e = xq - xr[u];
                        s[u] = fmaf(e, e, s[u]);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int p = p0 + u;
                    const float got = shfl_f32(wave_sum16(s[u]), ((lane - p * 4) & 3) * 16);
                    const int64_t jj = base + lane;
                    if (lane >= p * 4 && lane < p * 4 + 4 && jj < rend && jj != self)
                        cand = make_key(got, (uint32_t)jj);
                }
            }
            cand = seg_sort<64>(cand);
            list = seg_merge_sorted<64>(list, cand);
        }
        sl[wv][lane] = list;
        __syncthreads();
        if (wv == 0) {
            uint64_t a = sl[0][lane];
            for (int o = 1; o < 4; ++o) a = seg_merge_sorted<64>(a, sl[o][lane]);
            if (P == 1) write_row(row, a);
            else if (lane < kListW) lists[job * kListW + lane] = a;
        }
        __syncthreads();
    }
    if (P == 1 || (int64_t)blockIdx.x >= jobs) return;
    // P > 1: one job per workgroup; the last one merges (k <= kListW)
    if (threadIdx.x < 64) __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) order_ = atomicAdd(done, 1u);
    __syncthreads();
    if ((int64_t)order_ != jobs - 1) return;
    __threadfence();
    for (int64_t f = wv; f < cnt; f += 4) {
        // even parts in lanes 0..31, odd ones in lanes 32..63
        const int h = lane >> 5;
        uint64_t a = kEmptyList;
        for (int64_t c = 0; c < P; c += 2)
            a = seg_merge_sorted<32>(a, c + h < P ? lists[(f * P + c + h) * kListW + (lane & 31)] : kEmptyCand);
        const uint64_t rv = shfl_xor_u64(a, 31);
        write_row(fb_rows[f], seg_bitonic_merge<64>(h ? rv : a));
    }
}

// ------------------------------------------------------------------ host

template <int OUT>
static void launch_stage(const knn_matrix& X, void* Xs, int ldp, float* norms, unsigned* maxn,
                         const uint32_t* rowmap, int aux, hipStream_t st)
{
    dim3 grid((unsigned)std::min<int64_t>(ceil_div(X.n, 16), 4096)), block(256);
    switch (X.dtype) {
    case KNN_F32:
        stage_kernel<KNN_F32, OUT><<<grid, block, 0, st>>>(X.data, X.n, X.d, X.ld, Xs, ldp, norms, maxn, rowmap, aux);
        break;
    case KNN_BF16:
        stage_kernel<KNN_BF16, OUT><<<grid, block, 0, st>>>(X.data, X.n, X.d, X.ld, Xs, ldp, norms, maxn, rowmap, aux);
        break;
    default:
        stage_kernel<KNN_F16, OUT><<<grid, block, 0, st>>>(X.data, X.n, X.d, X.ld, Xs, ldp, norms, maxn, rowmap, aux);
        break;
    }
}

static void launch_stage_kind(int kind, const knn_matrix& X, void* Xs, int ldp, float* norms, unsigned* maxn,
                              const uint32_t* rowmap, int aux, hipStream_t st)
{
    if (kind == KNN_BF16) launch_stage<KNN_BF16>(X, Xs, ldp, norms, maxn, rowmap, aux, st);
    else if (kind == KNN_F16) launch_stage<KNN_F16>(X, Xs, ldp, norms, maxn, rowmap, aux, st);
    else launch_stage<KNN_F32>(X, Xs, ldp, norms, maxn, rowmap, aux, st);
}

// Staged copy of a matrix for the GEMM (FP32 ld = roundup(d, 32) or BF16 /
// FP16 ld = roundup(d, 64), both 128-byte multiples), norms and max norm.
// kind (KNN_F32, KNN_BF16, KNN_F16) is the staged element type; values are
// rounded to nearest even.  Row r of the copy is row rowmap[r] of X (rowmap
// nullable: identity).  With aux, ld leaves room for the two trailing FP32
// words (see stage_kernel).
knn_status stage_matrix(ScratchAlloc& ws, const knn_matrix& X, int kind, void** Xs, int* ldp,
                        float** norms, unsigned* maxnorm, hipStream_t st, const uint32_t* rowmap,
                        int aux)
{
    const bool half = kind != KNN_F32;
    const int64_t need = X.d + (aux ? (half ? 4 : 2) : 0);
    *ldp = half ? (int)round_up(need, 64) : (int)round_up(need, 32);
    knn_status r = ws.alloc(Xs, (size_t)X.n * (size_t)(*ldp) * (half ? 2 : 4));
    if (r != KNN_OK) return r;
    r = ws.alloc(norms, (size_t)X.n);
    if (r != KNN_OK) return r;
    launch_stage_kind(kind, X, *Xs, *ldp, *norms, maxnorm, rowmap, aux, st);
    KNN_HIP(hipGetLastError());
    return KNN_OK;
}

// Norms, largest norm (*maxn, zeroed beforehand) and staged rows of a matrix
// for the FP32 Gram.  kind: KNN_SPLIT or KNN_F16.  rmax: see split_kernel.
static void launch_full(int kind, const knn_matrix& X, void* Xs, int ldp, float* norms, unsigned* maxn,
                        const unsigned* rmax, hipStream_t st)
{
    const unsigned ng = (unsigned)std::min<int64_t>(ceil_div(X.n, 32), 4096);
    const unsigned sg = (unsigned)std::min<int64_t>(ceil_div(X.n * (ldp / 8), 256), 16384);
#define KNN_FULL(DT)                                                                                             \
    norm_kernel<DT><<<ng, 256, 0, st>>>(X.data, X.n, X.d, X.ld, norms, maxn);                                    \
    if (kind == KNN_SPLIT)                                                                                       \
        split_kernel<DT, KNN_SPLIT><<<sg, 256, 0, st>>>(X.data, X.n, X.d, X.ld, (_Float16*)Xs, ldp, maxn, rmax); \
    else                                                                                                         \
        split_kernel<DT, KNN_F16><<<sg, 256, 0, st>>>(X.data, X.n, X.d, X.ld, (_Float16*)Xs, ldp, maxn, rmax)
    if (X.dtype == KNN_F32) {
        KNN_FULL(KNN_F32);
    } else if (X.dtype == KNN_BF16) {
        KNN_FULL(KNN_BF16);
    } else {
        KNN_FULL(KNN_F16);
    }
#undef KNN_FULL
}

static knn_status stage_full(ScratchAlloc& ws, const knn_matrix& X, int kind, void** Xs, int* ldp, float** norms,
                             unsigned* maxn, hipStream_t st)
{
    *ldp = (int)round_up(X.d, kind == KNN_SPLIT ? 32 : 64);
    knn_status r = ws.alloc(Xs, (size_t)X.n * (size_t)(*ldp) * (kind == KNN_SPLIT ? 4 : 2));
    if (r != KNN_OK) return r;
    if ((r = ws.alloc(norms, (size_t)X.n)) != KNN_OK) return r;
    launch_full(kind, X, *Xs, *ldp, *norms, maxn, nullptr, st);
    KNN_HIP(hipGetLastError());
    return KNN_OK;
}

// Bound of a GEMM distance's error, in units of u (|q| + |r|)^2, u = 2^-24.
// One 32x32x16 FP16 MFMA adds 16 exact products to the incoming sum c; on
// gfx950 its result was measured within u (9 sum |products| + 2 |c|) of the
// exact value over products and sums of every relative magnitude (addends are
// aligned to the largest of their group and truncated, so a group of eight
// loses up to 7u of its largest), taken as 9 and 3.  Sampled: 8e8 outputs, products
// of normal, positive and cancelling factors over up to 2^28 in magnitude, sums from
// 2^-20 to 2^20 and the negated sum of the products, one dominant product with
// the rest around its truncation grid; the largest error was 1.005 of that
// expression, where c = 0.  So the 16 below, which counts the 9, leaves room:
// 13 in its place would still do.  A dot product of n instructions (three per 16 elements of split
// rows) whose sums stay below |q||r| is off by u (9 + 3 n) |q||r|, its parts'
// own rounding adds 12 u |q||r|, and the distance by twice the total,
// (1.5 n + 10.5) of (|q| + |r|)^2; scores sum from -|r|^2 / 2, with sums
// below |q||r| + |r|^2 / 2: 3 n.  Norms and the final sum: less than 3.
// Measured on the benchmark's data shapes, d = 17 .. 784: at most 11 (16 on
// the FP32 MFMA's own sums), rms 0.61 to 0.90 of the FP32 MFMA's error.  (Rows
// far below the common scale have the parts' absolute error besides; against the
// largest norm it is nothing, and merge_rerank_kernel's eabs and
// rank_tile_kernel's eabs stand for it where it is not.)
static float split_err(int d, int kind)
{
    const int64_t n = (kind == KNN_SPLIT ? 3 : 1) * ceil_div(d, 16);
    return 3.0f * (float)n + 16.0f;
}

// Zero n words (a fill kernel rather than hipMemsetAsync, so that no memset
// node is recorded when a caller captures the stream).
__global__ __launch_bounds__(64) void zero_words_kernel(unsigned* __restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 64) p[i] = 0u;
}

// Reference splits of a query chunk of qn rows: enough workgroups to fill
// the chip (about 2048), at most 4; every split starts from empty lists,
// which costs merges.
static int exact_splits(int64_t qn)
{
    const int64_t nblk = ceil_div(qn, kTileRows);
    const int64_t S = ceil_div(2048, nblk);
    return (int)(S < 1 ? 1 : (S > 4 ? 4 : S));
}

// Splits of the gated route, where a split costs no insertions: whole waves
// of the chip's resident slots (two workgroups on each of 256 CUs) to 90%, at
// least two tiles per split (2,000 x 300 FP32: 278 us at 2 splits, 149 at 8; one
// query in 2,000 x 784 BF16: 478 us with all 16 tiles in one workgroup, 135 at 8).
static int filling_splits(int64_t qn, int64_t nr)
{
    const int64_t nblk = ceil_div(qn, kTileRows), slots = 512;
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(16, ceil_div(nr, kTileRows) / 2));
    int best = 1;
    double fill = 0.0;
    for (int S = 1; S <= most; ++S) {
        const int64_t b = nblk * S;
        const double f = (double)b / (double)(ceil_div(b, slots) * slots);
        if (f > 1.02 * fill) {
            fill = f;
            best = S;
        }
        if (fill >= 0.9) break;
    }
    return best;
}

// Tiles of the gate's sample, for references of lds staged units.  A sample of
// m references costs m scores per row and leaves about 41 nr / m keys to
// append, each as much as some 320 / steps scores (steps: 128-byte chunks of a
// row): least in all at m = sqrt(13,200 nr / steps).  20,000 x 128 FP32 at 0.25,
// 0.5, 1, 2 times that: 671 / 640 / 670 / 794 us; 70,000 x 784 BF16 14.8 / 14.8 /
// 13.8 / 14.5 ms; 10,000 queries x 1M x 50 FP32 6.0 / 5.6 / 5.1 / 5.2 ms.
static int gate_tiles(int64_t nr, int lds)
{
    const double m = sqrt(13200.0 * (double)nr * 64.0 / (double)lds);
    return (int)std::min<int64_t>(ceil_div(nr, kTileRows), std::max<int64_t>(32, (int64_t)(m / kTileRows)));
}

static size_t elem_bytes(int dtype) { return dtype == KNN_F32 ? 4 : 2; }

// Scratch bytes of one exact call with query chunks of qc rows (every
// request rounded to 256 bytes, as the allocators carve them).
static size_t exact_scratch(const knn_matrix& Q, const knn_matrix& R, bool same, bool bf, int64_t qc)
{
    auto r256 = [](size_t b) { return (size_t)round_up((int64_t)(b ? b : 1), 256); };
    const int ldp = bf ? (int)round_up(R.d, 64) : (int)round_up(R.d, 32);
    const size_t eb = bf ? 2 : 4;
    size_t b = r256(16) + r256((size_t)R.n * ldp * eb) + r256((size_t)R.n * 4);
    if (!same) b += r256((size_t)qc * ldp * eb) + r256((size_t)qc * 4);
    const int S = exact_splits(qc);
    const int64_t slen = round_up(ceil_div(R.n, S), kTileRows);
    const int Sx = (int)ceil_div(R.n, slen);
    b += r256((size_t)qc * Sx * kListW * 8) + r256((size_t)qc * 4);
    return b;
}

// The exact k-NN of Q's rows among R's rows.  Queries are processed in
// chunks of qc rows (all of them when budget is 0) so that the scratch,
// taken from ws, stays within `budget` bytes: the staged reference set
// plus, per chunk, the staged query rows, the split lists and the fallback
// list.  A smaller budget means more chunks, each a pass over R: time for
// memory.  self_mode 1 excludes reference row q for query q (Q == R);
// self_mode 2 excludes q_self[q].
// The exact path for d <= kRankDirectD in FP32: direct canonical distances
// (exact_direct_kernel) over S reference splits, merged by
// merge_rerank_kernel without a certificate (the lists are canonical).
// Scratch: the split lists, S * kListW * 8 bytes per query row of a chunk.
template <int DT>
static void launch_exact_direct(int dc, int km, dim3 grid, hipStream_t st, const void* Qd, int64_t ldq,
                                int64_t nq, const knn_matrix& R, const int32_t* qself, int self_mode,
                                int64_t q0, int k, int64_t split_len, int S, uint64_t* part)
{
#define KNN_ED(DC, KM)                                                                                 \
    exact_direct_kernel<DT, DC, KM><<<grid, 256, 0, st>>>(Qd, ldq, nq, R.data, R.ld, R.n, R.d, qself,  \
                                                          self_mode, q0, k, split_len, S, part)
    if (km == 16) {
        if (dc == 2) KNN_ED(2, 16);
        else if (dc == 3) KNN_ED(3, 16);
        else KNN_ED(0, 16);
    } else {
        if (dc == 2) KNN_ED(2, 32);
        else if (dc == 3) KNN_ED(3, 32);
        else KNN_ED(0, 32);
    }
#undef KNN_ED
}

static knn_status exact_direct_impl(const knn_matrix& Q, const knn_matrix& R, const int32_t* q_self,
                                    int self_mode, int32_t k, int32_t out_kind, int32_t* out_idx,
                                    float* out_dist, hipStream_t st, ScratchAlloc& ws, int64_t budget)
{
    const int64_t nblk = ceil_div(Q.n, 256);
    int S = (int)std::min<int64_t>(16, std::max<int64_t>(1, ceil_div(2048, nblk)));
    S = (int)std::min<int64_t>(S, ceil_div(R.n, 256));
    const int64_t split_len = round_up(ceil_div(R.n, S), 256);
    S = (int)ceil_div(R.n, split_len);
    const size_t per_row = (size_t)S * kListW * 8;
    int64_t qc = Q.n;
    if (budget > 0 && (size_t)round_up((int64_t)(qc * per_row), 256) > (size_t)budget) {
        qc = (budget / (int64_t)per_row) / 256 * 256;
        if (qc < 256)
            return fail(KNN_ENOMEM, "workspace limit of " + std::to_string(budget) + " bytes is below the " +
                                        std::to_string(256 * per_row) + " bytes one 256-query chunk needs");
    }
    uint64_t* part = nullptr;
    knn_status r = ws.alloc(&part, (size_t)qc * S * kListW);
    if (r != KNN_OK) return r;
    const int km = k <= 16 ? 16 : 32;
    const int dc = R.d == 2 || R.d == 3 ? R.d : 0;
    const size_t qeb = elem_bytes(Q.dtype);
    for (int64_t q0 = 0; q0 < Q.n; q0 += qc) {
        const int64_t nq = Q.n - q0 < qc ? Q.n - q0 : qc;
        const void* Qd = (const char*)Q.data + (size_t)q0 * Q.ld * qeb;
        const int32_t* qself = self_mode == 2 ? q_self + q0 : nullptr;
        const dim3 grid((unsigned)ceil_div(nq, 256), (unsigned)S);
        if (Q.dtype == KNN_F32)
            launch_exact_direct<KNN_F32>(dc, km, grid, st, Qd, Q.ld, nq, R, qself, self_mode, q0, k, split_len, S, part);
        else if (Q.dtype == KNN_BF16)
            launch_exact_direct<KNN_BF16>(dc, km, grid, st, Qd, Q.ld, nq, R, qself, self_mode, q0, k, split_len, S,
                                          part);
        else
            launch_exact_direct<KNN_F16>(dc, km, grid, st, Qd, Q.ld, nq, R, qself, self_mode, q0, k, split_len, S,
                                         part);
        KNN_HIP(hipGetLastError());
        int32_t* oi = out_idx + q0 * k;
        float* od = out_dist + q0 * k;
        const dim3 mgrid((unsigned)ceil_div(nq, 4));
#define KNN_MR(DT)                                                                                       \
    merge_rerank_kernel<DT><<<mgrid, 256, 0, st>>>(part, nullptr, nullptr, 0, 0, nullptr, S, nq, k, k, Qd, Q.ld, \
                                                   R.data, R.ld, R.d, nullptr,                                  \
                                                   nullptr, 0.0f, 0.0f, 0.0f, 0, 0, out_kind, oi, od, nullptr, nullptr)
        if (Q.dtype == KNN_F32) KNN_MR(KNN_F32);
        else if (Q.dtype == KNN_BF16) KNN_MR(KNN_BF16);
        else KNN_MR(KNN_F16);
#undef KNN_MR
        KNN_HIP(hipGetLastError());
    }
    return KNN_OK;
}

// The tile pass of one query chunk, or (gated) the gate and the gated pass.
struct TileArgs {
    const void* Qs;
    const float* qn;
    int64_t nq;
    const void* Rs;
    const float* rn;
    int64_t nr;
    int ld;
    const int32_t* qself;
    int self_mode;
    int64_t q0;
    int kp;
    int64_t split_len;
    int S;
    const unsigned *rmax, *qmax;
    uint64_t* part;
    bool gated;
    int ntiles;       // the gate's sample
    float gate_err, cert_err;   // cert_err 0: no certificate
    float* lims;
    uint32_t* cnt;
};

template <int OUT, bool ARES>
static void launch_tiles_a(const TileArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)ceil_div(a.nq, kTileRows), (unsigned)a.S);
    if (!a.gated) {
        exact_tile_kernel<OUT, ARES><<<grid, 256, 0, st>>>(a.Qs, a.qn, a.nq, a.Rs, a.rn, a.nr, a.ld, a.qself,
                                                           a.self_mode, a.q0, a.kp, a.split_len, a.S, a.rmax, a.qmax,
                                                           a.part);
        return;
    }
    // the group scores fit in the buffers they precede (32 floats per split)
    float* gtop = (float*)a.part;
    const dim3 ggrid(grid.x, (unsigned)std::min(a.S, a.ntiles));
    exact_gate_kernel<OUT, ARES><<<ggrid, 256, 0, st>>>(a.Qs, a.nq, a.Rs, a.rn, a.nr, a.ld, a.qself, a.self_mode, a.q0,
                                                        a.ntiles, a.rmax, a.qmax, gtop);
    gate_select_kernel<<<(unsigned)ceil_div(a.nq, 8), 256, 0, st>>>(gtop, a.nq, (int)ggrid.y, a.kp, a.qn, a.rmax,
                                                                    a.qmax, a.gate_err, a.cert_err, a.lims);
    exact_append_kernel<OUT, ARES><<<grid, 256, 0, st>>>(a.Qs, a.qn, a.nq, a.Rs, a.rn, a.nr, a.ld, a.qself,
                                                         a.self_mode, a.q0, a.kp, a.split_len, a.S, a.rmax, a.qmax,
                                                         a.lims, a.part, a.cnt);
}

template <int OUT>
static void launch_tiles(bool ares, const TileArgs& a, hipStream_t st)
{
    if (ares) launch_tiles_a<OUT, true>(a, st);
    else launch_tiles_a<OUT, false>(a, st);
}

static knn_status exact_impl(const knn_matrix& Q, const knn_matrix& R, bool same,
                             const int32_t* q_self, int self_mode, int32_t k, int32_t precision,
                             int32_t rerank_k, int32_t out_kind, int32_t* out_idx, float* out_dist,
                             hipStream_t st, ScratchAlloc& ws, int64_t budget)
{
    if (precision != KNN_PREC_FP32 && precision != KNN_PREC_BF16 && precision != KNN_PREC_FP16)
        return fail(KNN_EINVAL, "precision must be KNN_PREC_FP32, KNN_PREC_BF16 or KNN_PREC_FP16");
    if (out_kind != KNN_OUT_L2 && out_kind != KNN_OUT_SQL2)
        return fail(KNN_EINVAL, "out_kind must be KNN_OUT_L2 or KNN_OUT_SQL2");
    if (!out_idx || !out_dist) return fail(KNN_EINVAL, "null output pointer");
    const int64_t avail = R.n - (self_mode ? 1 : 0);   // candidates per query
    if (k < 1 || (int64_t)k > avail) return fail(KNN_EINVAL, "k must satisfy 1 <= k <= number of candidates");
    int kp = rerank_k;
    if (kp == 0) kp = 2 * k < kListW ? 2 * k : kListW;
    if (kp < k) return fail(KNN_EINVAL, "rerank_k must be >= k");
    if (kp > kListW || k > KNN_MAX_K)
        return fail(KNN_ENOTSUP, "rerank_k and k above 32 are not supported by the exact path");
    if (budget < 0) return fail(KNN_EINVAL, "workspace limit must be >= 0");
    if (Q.n == 0) return KNN_OK;
    // staged element kind: the 16-bit type of the MFMA form; in FP32, split
    // FP16 pairs, or one FP16 value for 16-bit inputs (whose low part is 0)
    const bool full = precision == KNN_PREC_FP32;
    const int kind = precision == KNN_PREC_BF16 ? KNN_BF16
                     : full && R.dtype == KNN_F32 ? KNN_SPLIT : KNN_F16;
    const bool bf = !full;
    // a few coordinates: exact_direct_kernel's launches are cheaper sooner (1500 x 2
    // 61 us against 78, 2000 x 2 73 against 75, 3000 x 2 108 against 77; 2000 x 8 72
    // against 115, 3000 x 8 109 against 119), and its work per pair is less (queries x
    // references x coordinates: 4000 x 1000 x 2 67 us against 78, 4000 x 1500 x 2 83
    // and 79, 16,000 x 600 x 2 122 and 85; 4000 x 2500 x 8 113 and 122, 16,000 x 1000 x
    // 8 155 and 131, 100,000 x 100 x 8 199 and 164)
    const int64_t small_refs = R.d > kRankDirectD ? kSmallRefs : (R.d > kLowdimD ? 2560 : 1536);
    const double small_pairs = R.d > kRankDirectD ? kSmallWork / (6.0 * R.d + 150.0) : (R.d > kLowdimD ? 1.1e7 : 5e6);
    const bool small = full && R.n <= small_refs &&
                       (double)Q.n * (double)(R.n + (R.d > kRankDirectD ? 0 : 64)) <= small_pairs;
    if (full && R.d <= kRankDirectD && !(small && budget == 0)) {
        // the pruned search needs eleven launches (3000 x 3 88 us against 76,
        // 5000 x 3 96 against 115; one query in 4000 x 2 73 against 64, in 20,000 x 2
        // 79 against 160); under a workspace limit the other one, which can be cut up
        if (R.d <= kLowdimD && budget == 0 && R.n >= 6144)
            return lowdim_knn(Q, R, same, q_self, self_mode, k, out_kind, out_idx, out_dist, st, ws);
        return exact_direct_impl(Q, R, q_self, self_mode, k, out_kind, out_idx, out_dist, st, ws, budget);
    }

    // query chunk: the largest multiple of the tile height that fits
    int64_t qc = Q.n;
    if (budget > 0 && exact_scratch(Q, R, same, bf, qc) > (size_t)budget) {
        int64_t lo = 0, hi = ceil_div(Q.n, kTileRows);   // in tiles: lo fits (0 = none), hi does not
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) / 2;
            if (exact_scratch(Q, R, same, bf, mid * kTileRows) <= (size_t)budget) lo = mid;
            else hi = mid;
        }
        if (lo == 0)
            return fail(KNN_ENOMEM, "workspace limit of " + std::to_string(budget) + " bytes is below the " +
                                        std::to_string(exact_scratch(Q, R, same, bf, kTileRows)) +
                                        " bytes the staged reference set and one 128-query chunk need");
        qc = lo * kTileRows;
    }
    if (small) {
        // Few queries leave CUs idle: four waves share one (100 queries in 1,000 /
        // 4,000 x 50: 45 / 92 us, 57 / 135 with a wave each; 300: 66 / 159 and
        // 58 / 136, for then two workgroups of 256 registers meet on a CU).
        const bool wide = Q.n <= 256 && R.n >= 512;
        const unsigned g = (unsigned)(wide ? Q.n : ceil_div(Q.n, 4));
#define KNN_SM(DT, WQ)                                                                                           \
    exact_small_kernel<DT, WQ><<<g, 256, 0, st>>>(Q.data, Q.ld, (int)Q.n, R.data, R.ld, (int)R.n, R.d, q_self,     \
                                                  self_mode, k, out_kind, out_idx, out_dist)
        if (Q.dtype == KNN_F32) {
            if (wide) KNN_SM(KNN_F32, 4);
            else KNN_SM(KNN_F32, 1);
        } else if (Q.dtype == KNN_BF16) {
            if (wide) KNN_SM(KNN_BF16, 4);
            else KNN_SM(KNN_BF16, 1);
        } else {
            if (wide) KNN_SM(KNN_F16, 4);
            else KNN_SM(KNN_F16, 1);
        }
#undef KNN_SM
        KNN_HIP(hipGetLastError());
        KNN_HIP(hipStreamSynchronize(st));
        return KNN_OK;
    }
    // the gated route's buffers (below): at most 1 GiB per query chunk
    if (budget == 0) qc = std::min<int64_t>(qc, 4096 * kTileRows);

    knn_status r;
    // [0] = max ref norm bits, [1] = fallback count, [2] = fallback parts done,
    // [3] = max query norm bits (FP32, Q != R)
    unsigned* words = nullptr;
    r = ws.alloc(&words, 4);
    if (r != KNN_OK) return r;
    zero_words_kernel<<<1, 64, 0, st>>>(words, 4);
    void *Rs = nullptr, *Qb = nullptr;
    float *rn = nullptr, *qnb = nullptr;
    int ldp = 0;
    if (full) r = stage_full(ws, R, kind, &Rs, &ldp, &rn, words, st);
    else r = stage_matrix(ws, R, kind, &Rs, &ldp, &rn, words, st, nullptr, 0);
    if (r != KNN_OK) return r;
    const size_t eb = kind == KNN_SPLIT ? 4 : 2;
    if (!same) {
        if ((r = ws.alloc(&Qb, (size_t)qc * ldp * eb)) != KNN_OK) return r;
        if ((r = ws.alloc(&qnb, (size_t)qc)) != KNN_OK) return r;
    }
    // row stride in staged units (a split element is two)
    const int lds = kind == KNN_SPLIT ? 2 * ldp : ldp;
    const bool ares = lds <= (kind == KNN_SPLIT ? TileCfg<KNN_SPLIT>::AMAX : TileCfg<KNN_F16>::AMAX);
    // the gated route needs 2 KiB of scratch per row and split: not under a
    // limit; with two to four tiles of long rows its second pass over the
    // products costs more than the insertions (500 x 784 BF16: 187 us against 142;
    // 500 x 200: 105 and 110, 128 x 784: 105 and 140, 100,000 queries in 500 x 200:
    // 503 and 881); one to four queries in few references insert little (BF16, one
    // in 1,000 x 50: 63 us against 53, in 4,000 x 50 80 and 75, in 6,000 x 50 86 and
    // 87; four in 1,000 x 50 65 and 72, x 784 135 and 123)
    const bool few = Q.n <= 4 && Q.n * R.n <= 4096;
    bool gated = budget == 0 && !few && (ares || lds <= 256 || R.n <= kTileRows || R.n > 4 * kTileRows);
    int64_t split_len = 0;
    int S = 0;
    uint64_t* part = nullptr;
    auto buffers = [&]() {
        const int S0 = gated ? filling_splits(qc, R.n) : exact_splits(qc);
        split_len = round_up(ceil_div(R.n, S0), kTileRows);
        S = (int)ceil_div(R.n, split_len);
        return ws.alloc(&part, (size_t)qc * S * (gated ? kCandCap : kListW));
    };
    const std::string before = last_error();
    r = buffers();
    if (r == KNN_ENOMEM && gated) {
        // a device nearly full: the lists take an eighth and at most four splits
        gated = false;
        if ((r = buffers()) == KNN_OK) set_error(before);
    }
    if (r != KNN_OK) return r;
    int32_t* fb_rows = nullptr;
    r = ws.alloc(&fb_rows, (size_t)qc);
    if (r != KNN_OK) return r;
    float* lims = nullptr;
    uint32_t* cnt = nullptr;
    int ntiles = 0;
    if (gated) {
        if ((r = ws.alloc(&lims, (size_t)qc)) != KNN_OK) return r;
        if ((r = ws.alloc(&cnt, (size_t)qc * S)) != KNN_OK) return r;
        ntiles = gate_tiles(R.n, lds);
    }

    // GEMM error bound (FP32): split_err u (|q| + max|r|)^2 with u = 2^-24;
    // re-rank bound: (d/16 + 8) u relative.
    const float u = 5.9604645e-08f;
    const float err_coef = split_err(R.d, kind) * u * 1.01f;
    const float edir = (float)(R.d / 16 + 8) * u, eabs = 2.0f * u * sqrtf((float)R.d);
    const int certify = bf ? 0 : 1;
    int* fb_count = (int*)(words + 1);
    const size_t qeb = elem_bytes(Q.dtype);

    for (int64_t q0 = 0; q0 < Q.n; q0 += qc) {
        const int64_t nq = Q.n - q0 < qc ? Q.n - q0 : qc;
        const void* Qs;
        const float* qn;
        if (q0 > 0) zero_words_kernel<<<1, 64, 0, st>>>(words + 1, 3);
        if (same) {
            Qs = (const char*)Rs + (size_t)q0 * ldp * eb;
            qn = rn + q0;
        } else {
            const knn_matrix Qc = {(const char*)Q.data + (size_t)q0 * Q.ld * qeb, nq, Q.d, Q.ld, Q.dtype};
            if (full) launch_full(kind, Qc, Qb, ldp, qnb, words + 3, words, st);
            else launch_stage_kind(kind, Qc, Qb, ldp, qnb, nullptr, nullptr, 0, st);
            Qs = Qb;
            qn = qnb;
        }
        const int32_t* qself = self_mode == 2 ? q_self + q0 : nullptr;
        
        const unsigned* qmax = !full ? nullptr : (same ? words : words + 3);
        const TileArgs ta = {Qs, qn, nq, Rs, rn, R.n, lds, qself, self_mode, q0, kp, split_len, S, words, qmax, part,
                             gated, ntiles, 2.0f * split_err(R.d, kind) * u, certify ? err_coef : 0.0f, lims, cnt};
        if (kind == KNN_BF16) launch_tiles<KNN_BF16>(ares, ta, st);
        else if (kind == KNN_F16) launch_tiles<KNN_F16>(ares, ta, st);
        else launch_tiles<KNN_SPLIT>(ares, ta, st);
        KNN_HIP(hipGetLastError());

        const void* Qd = (const char*)Q.data + (size_t)q0 * Q.ld * qeb;
        int32_t* oi = out_idx + q0 * k;
        float* od = out_dist + q0 * k;
        dim3 mgrid((unsigned)ceil_div(nq, 4));
#define KNN_MR(DT)                                                                              \
    merge_rerank_kernel<DT><<<mgrid, 256, 0, st>>>(part, cnt, qself, self_mode, q0, qmax, S, nq, kp, k, Qd, Q.ld, R.data, R.ld,  \
                                                   R.d, qn, words, err_coef, edir, eabs, certify, \
                                                   avail, out_kind, oi, od, fb_rows, fb_count)
        if (Q.dtype == KNN_F32) KNN_MR(KNN_F32);
        else if (Q.dtype == KNN_BF16) KNN_MR(KNN_BF16);
        else KNN_MR(KNN_F16);
#undef KNN_MR
        KNN_HIP(hipGetLastError());
        if (certify) {
            dim3 fgrid(1024);
#define KNN_FB(DT)                                                                              \
    exact_fallback_kernel<DT><<<fgrid, 256, 0, st>>>(fb_rows, fb_count, Qd, Q.ld, R.data, R.ld, \
                                                     R.n, R.d, qself, self_mode, q0, k,         \
                                                     out_kind, oi, od, part, nq * S, words + 2)
            if (Q.dtype == KNN_F32) KNN_FB(KNN_F32);
            else if (Q.dtype == KNN_BF16) KNN_FB(KNN_BF16);
            else KNN_FB(KNN_F16);
#undef KNN_FB
            KNN_HIP(hipGetLastError());
        }
    }
    KNN_HIP(hipStreamSynchronize(st));
    return KNN_OK;
}

// ------------------------------------------------------------ quality

// One wave per row i.  N(i) (row i of Hn, the exact lists in X) sits in
// lanes 0..k-1, L(i) (row i of Ln, the lists in the embedding Y) likewise.
// U = L \ N are the trustworthiness probes: their canonical FP32 distances
// in X as keys; V = N \ L the continuity probes, keyed by their distances in
// Y.  Both are sorted ascending and padded with kEmptyCand to kRankP (k <=
// kRankP); hits[i] = |N intersect L|.  With all_l, U is all of L (N is not
// needed; Hn may be null).  pu, pv and hits may each be null: that output
// is not formed.
__global__ __launch_bounds__(256) void quality_probes_kernel(int64_t n, int k, const int32_t* __restrict__ Hn,
                                                             const int32_t* __restrict__ Ln,
                                                             const float* __restrict__ Xs, int ldx, int dx,
                                                             const float* __restrict__ Ys, int ldy, int dy,
                                                             uint64_t* __restrict__ pu, uint64_t* __restrict__ pv,
                                                             int32_t* __restrict__ hits, int all_l)
{
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= n) return;   // uniform across the wave
    const int32_t hv = lane < k && Hn ? Hn[i * k + lane] : -1;
    const int32_t lv = lane < k ? Ln[i * k + lane] : -1;
    bool l_in_n = false, n_in_l = false;
    for (int r = 0; r < k; ++r) {
        // lane r's entries by readlane, outside any lane-dependent branch
        const int32_t hr = (int32_t)bcast_u32((uint32_t)hv, r), lr = (int32_t)bcast_u32((uint32_t)lv, r);
        l_in_n |= lv == hr;
        n_in_l |= hv == lr;
    }
    // all_l: every member of L(i) is a probe in X (no N(i) yet); a member
    // of N(i) then has rank <= k and adds nothing to the trust sum.  A side
    // whose output is null computes nothing; without Hn there is no V side
    const bool inU = pu && lane < k && (all_l || !l_in_n), inV = Hn && lane < k && !n_in_l;
    const float du = dist_batch16<KNN_F32, 4>(Xs, ldx, i, (uint32_t)lv, inU, dx);
    const float dv = dist_batch16<KNN_F32, 4>(Ys, ldy, i, (uint32_t)hv, inV, dy);
    uint64_t ku = inU ? make_key(du, (uint32_t)lv) : kEmptyCand;
    uint64_t kv = inV ? make_key(dv, (uint32_t)hv) : kEmptyCand;
    ku = seg_sort<16>(ku);
    kv = seg_sort<16>(kv);
    if (lane < kRankP) {
        if (pu) pu[i * kRankP + lane] = ku;
        if (pv) pv[i * kRankP + lane] = kv;
    }
    const int nv = popc64(ballot(inV));
    if (hits && lane == 0) hits[i] = k - nv;   // |N & L| = k - |N \ L|
}

// Per row: trust = sum over U of (rank - k) = sum of (count + 1 - k), cont
// likewise over V; the three totals by exact integer atomics (order-free).
__global__ __launch_bounds__(256) void quality_reduce_kernel(int64_t n, int k, const uint64_t* __restrict__ pu,
                                                             const uint32_t* __restrict__ cu,
                                                             const uint64_t* __restrict__ pv,
                                                             const uint32_t* __restrict__ cv,
                                                             const int32_t* __restrict__ hits,
                                                             int64_t* __restrict__ trust_row,
                                                             int64_t* __restrict__ cont_row,
                                                             unsigned long long* __restrict__ tot)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long t = 0, c = 0, hsum = 0;
    if (i < n) {
        for (int p = 0; p < kRankP; ++p) {
            // rank - k where the rank exceeds k (probes of rank <= k, members
            // of both lists, add nothing)
            const uint32_t ru = cu[i * kRankP + p] + 1u, rv = cv[i * kRankP + p] + 1u;
            if (pu[i * kRankP + p] != kEmptyCand && ru > (uint32_t)k) t += (unsigned long long)(ru - (uint32_t)k);
            if (pv[i * kRankP + p] != kEmptyCand && rv > (uint32_t)k) c += (unsigned long long)(rv - (uint32_t)k);
        }
        hsum = (unsigned long long)hits[i];
        if (trust_row) trust_row[i] = (int64_t)t;
        if (cont_row) cont_row[i] = (int64_t)c;
    }
    for (int o = 32; o > 0; o >>= 1) {
        t += shfl_u64(t, (threadIdx.x & 63) ^ o);
        c += shfl_u64(c, (threadIdx.x & 63) ^ o);
        hsum += shfl_u64(hsum, (threadIdx.x & 63) ^ o);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&tot[0], hsum);
        atomicAdd(&tot[1], t);
        atomicAdd(&tot[2], c);
    }
}

static knn_status quality_impl(const knn_matrix& X, const knn_matrix& Y, int k, int32_t* hits_out,
                               int64_t* trust_out, int64_t* cont_out, double* metrics, hipStream_t st)
{
    const int64_t n = X.n;
    Workspace ws(st, 0);
    knn_status r;
    int32_t *Hn, *Ln, *hits;
    float *Hd, *Ld;
    if ((r = ws.alloc(&Hn, (size_t)n * k)) != KNN_OK) return r;
    if ((r = ws.alloc(&Ln, (size_t)n * k)) != KNN_OK) return r;
    if ((r = ws.alloc(&Hd, (size_t)n * k)) != KNN_OK) return r;
    if ((r = ws.alloc(&Ld, (size_t)n * k)) != KNN_OK) return r;
    // exact lists in both spaces (FP32, canonical re-rank).  Above
    // kRankDirectD dimensions X's lists come from its rank pass (fused):
    // the same Gram tiles give the ranks and the split lists
    const bool fused = X.d > kRankDirectD;
    if ((r = exact_impl(Y, Y, true, nullptr, 1, k, KNN_PREC_FP32, 0, KNN_OUT_SQL2, Ln, Ld, st, ws, 0)) != KNN_OK)
        return r;
    if (!fused &&
        (r = exact_impl(X, X, true, nullptr, 1, k, KNN_PREC_FP32, 0, KNN_OUT_SQL2, Hn, Hd, st, ws, 0)) != KNN_OK)
        return r;
    unsigned* small;   // [0] max norm of X, [1] max norm of Y; then three u64 totals
    if ((r = ws.alloc(&small, 8)) != KNN_OK) return r;
    zero_words_kernel<<<1, 64, 0, st>>>(small, 8);
    void *Xs, *Ys;
    float *xn, *yn;
    int ldx, ldy;
    if ((r = stage_matrix(ws, X, KNN_F32, &Xs, &ldx, &xn, small, st, nullptr, 0)) != KNN_OK) return r;
    if ((r = stage_matrix(ws, Y, KNN_F32, &Ys, &ldy, &yn, small + 1, st, nullptr, 0)) != KNN_OK) return r;
    uint64_t *pu, *pv;
    uint32_t *cu, *cv;
    if ((r = ws.alloc(&pu, (size_t)n * kRankP)) != KNN_OK) return r;
    if ((r = ws.alloc(&pv, (size_t)n * kRankP)) != KNN_OK) return r;
    if ((r = ws.alloc(&cu, (size_t)n * kRankP)) != KNN_OK) return r;
    if ((r = ws.alloc(&cv, (size_t)n * kRankP)) != KNN_OK) return r;
    hits = hits_out;
    if (!hits && (r = ws.alloc(&hits, (size_t)n)) != KNN_OK) return r;
    // X's probes: L(i) \ N(i), or every member of L(i) when N(i) is not
    // known yet (fused); Y's probes N(i) \ L(i) and |N & L| once it is
    if (fused)
        quality_probes_kernel<<<(unsigned)ceil_div(n, 4), 256, 0, st>>>(n, k, nullptr, Ln, (const float*)Xs, ldx,
                                                                        X.d, (const float*)Ys, ldy, Y.d, pu, nullptr,
                                                                        nullptr, 1);
    else
        quality_probes_kernel<<<(unsigned)ceil_div(n, 4), 256, 0, st>>>(n, k, Hn, Ln, (const float*)Xs, ldx, X.d,
                                                                        (const float*)Ys, ldy, Y.d, pu, pv, hits, 0);
    KNN_HIP(hipGetLastError());
    const float u = 5.9604645e-08f;
    // The tile pass: S reference splits, so that the workgroups fill the
    // chip's resident slots (two per CU) in nearly whole waves; each
    // workgroup holds a queue of undecided pairs of one tile, launches of at
    // most kRankBlocks workgroups.
    int dev = 0, ncu = 256;
    KNN_HIP(hipGetDevice(&dev));
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1) ncu = 256;
    const int64_t nblk = ceil_div(n, kTileRows), ntile = nblk, slots = 2 * (int64_t)ncu;
    int S = 1;
    for (; S < kRankMaxSplits; ++S) {
        const int64_t b = nblk * S;   // stop once the waves of resident workgroups are 90% full on average
        if (b % slots == 0 || (double)b / (double)slots >= 0.9 * (double)ceil_div(b, slots)) break;
    }
    if (S > ntile) S = (int)ntile;
    const int64_t split_len = ceil_div(ntile, S) * kTileRows;
    S = (int)ceil_div(n, split_len);   // no empty split
    const int kp = 2 * k < kListW ? 2 * k : kListW;   // the lists' re-rank width, as knn_exact's default
    // scratch of one launch of query blocks: queues, and with lists the gates,
    // buffers, counts and the rows without a certificate
    int64_t per_launch = 0, lrows = 0;   // query blocks per launch, and their rows
    uint64_t *rq = nullptr, *part = nullptr;
    float* lims = nullptr;
    uint32_t* cnt = nullptr;
    int32_t* fb_rows = nullptr;
    unsigned* fb_count = nullptr;   // [1]: fallback parts done
    const std::string before = last_error();
    for (int64_t most = kRankBlocks / S;; most /= 2) {
        per_launch = most;
        lrows = std::min<int64_t>(nblk, per_launch) * kTileRows;
        const size_t queue = X.d > kRankDirectD || Y.d > kRankDirectD ? (size_t)(lrows / kTileRows) * S * kRankQueue : 0;
        const size_t cand = fused ? (size_t)lrows * S * kCandCap : 0;
        if (queue + cand == 0) break;
        r = ws.alloc(&rq, queue + cand);
        if (r == KNN_OK) set_error(before);
        if (r == KNN_OK || most < 2) break;
        // a device nearly full: fewer query blocks per launch
    }
    if (r != KNN_OK) return r;
    if (fused) {
        part = rq + (size_t)(lrows / kTileRows) * S * kRankQueue;
        if ((r = ws.alloc(&lims, (size_t)lrows)) != KNN_OK) return r;
        if ((r = ws.alloc(&cnt, (size_t)lrows * S)) != KNN_OK) return r;
        if ((r = ws.alloc(&fb_rows, (size_t)lrows)) != KNN_OK) return r;
        if ((r = ws.alloc(&fb_count, 2)) != KNN_OK) return r;
    }
    // ranks of the probes pz of Z's rows (FP32 rows Zf, norms zn, largest norm
    // mx) among Z's rows into cz; with lists also X's exact neighbours into Hn
    auto rank_tile = [&](const float* Zf, const float* zn, int ldf, int dz, const uint64_t* pz, const unsigned* mx,
                         uint32_t* cz, bool lists) -> knn_status {
        const int lds = 2 * (int)round_up(dz, 32);   // split rows, in FP16 values
        _Float16* Zs = nullptr;
        if ((r = ws.alloc((void**)&Zs, (size_t)n * lds * 2)) != KNN_OK) return r;
        split_kernel<KNN_F32, KNN_SPLIT><<<(unsigned)std::min<int64_t>(ceil_div(n * (lds / 16), 256), 16384), 256, 0, st>>>(
            Zf, n, dz, ldf, Zs, lds / 2, mx, nullptr);
        // Error of a GEMM distance: 2 |q||r| (9 + 3 i + s + 12 + 4) u with i
        // instructions per segment and s segments (see split_err: products and
        // running sums of a segment; the segments' additions; the parts' rounding;
        // the score's subtraction and slack), plus 4u (|q|^2 + |r|^2 + the
        // probe's distance) for the norms (FP64 sums rounded once) and the
        // probes' scores; the canonical distance's own error is edir.
        // The parts of elements far below the common scale are off by up to
        // 2^-25 of a scaled unit each, which no relative term covers: a score by
        // 2^-25 sqrt(d) (|q| + |r|) + d 2^-50 in scaled units.  Twice the first
        // is taken (eabs), and d 2^-24 for the second and for norms and
        // distances among FP32's denormals (eden).  Next to nothing for rows of
        // like norms; with one row 10^6 times the others the slack is some
        // 60 times as wide, from 10^8 times on most pairs are rechecked.
        const int chunks = lds / 64;
        const float inst = 6.0f * (float)std::min(chunks, kSegChunks), segs = (float)ceil_div(chunks, kSegChunks);
        const float ecd = 2.0f * (25.0f + 3.0f * inst + segs) * u * 1.01f, ecn = 4.04f * u;
        const float ed = (float)(dz / 16 + 8) * u, ea = u * sqrtf((float)dz), en = u * (float)dz;
        const bool ares = lds <= TileCfg<KNN_SPLIT>::AMAX;
        zero_words_kernel<<<(unsigned)std::min<int64_t>(ceil_div(n * kRankP, 64), 4096), 64, 0, st>>>(cz,
                                                                                                 n * kRankP);
        const int ntiles = gate_tiles(n, lds);
        const float err_coef = split_err(dz, KNN_SPLIT) * u * 1.01f;
        for (int64_t q0 = 0; q0 < n; q0 += per_launch * kTileRows) {
            const int64_t nq = std::min<int64_t>(n - q0, per_launch * kTileRows);
            const unsigned nb = (unsigned)ceil_div(nq, kTileRows);
            if (lists) {
                const dim3 gg(nb, (unsigned)std::min(S, ntiles));
                float* gtop = (float*)part;
                if (ares)
                    exact_gate_kernel<KNN_SPLIT, true><<<gg, 256, 0, st>>>(Zs + q0 * lds, nq, Zs, zn, n, lds, nullptr, 1,
                                                                           q0, ntiles, mx, mx, gtop);
                else
                    exact_gate_kernel<KNN_SPLIT, false><<<gg, 256, 0, st>>>(Zs + q0 * lds, nq, Zs, zn, n, lds, nullptr, 1,
                                                                            q0, ntiles, mx, mx, gtop);
                gate_select_kernel<<<(unsigned)ceil_div(nq, 8), 256, 0, st>>>(
                    gtop, nq, (int)gg.y, kp, zn + q0, mx, mx, 2.0f * split_err(dz, KNN_SPLIT) * u, err_coef, lims);
            }
#define KNN_RANK(L, A, NP)                                                                                        \
    rank_tile_kernel<L, A, NP><<<nb * (unsigned)S, 256, 0, st>>>(                                                  \
        Zs + q0 * lds, zn + q0, nq, Zs, zn, n, lds, Zf + q0 * ldf, Zf, ldf, dz, q0, pz + q0 * kRankP, mx, ecd, ecn, \
        ed, ea, en, S, split_len, cz + q0 * kRankP, rq, kp, lims, part, cnt)
#define KNN_RANK_NP(L, A)                                                                                         \
    if (k <= 8) KNN_RANK(L, A, 8);                                                                                \
    else if (k <= 12) KNN_RANK(L, A, 12);                                                                         \
    else KNN_RANK(L, A, 16)
            if (lists && ares) {
                KNN_RANK_NP(true, true);
            } else if (lists) {
                KNN_RANK_NP(true, false);
            } else if (ares) {
                KNN_RANK_NP(false, true);
            } else {
                KNN_RANK_NP(false, false);
            }
#undef KNN_RANK_NP
#undef KNN_RANK
            rank_wide_kernel<<<(unsigned)std::min<int64_t>(nq, 4096), 256, 0, st>>>(Zf, ldf, dz, q0, nq, n, pz + q0 * kRankP,
                                                                                  mx, cz + q0 * kRankP);
            KNN_HIP(hipGetLastError());
            if (!lists) continue;
            // X's exact lists: merge, canonical re-rank, certificate, and the
            // exhaustive search for rows not certified
            zero_words_kernel<<<1, 64, 0, st>>>(fb_count, 2);
            const void* Xq = (const char*)X.data + (size_t)q0 * X.ld * elem_bytes(X.dtype);
#define KNN_QMR(DT)                                                                                              \
    merge_rerank_kernel<DT><<<(unsigned)ceil_div(nq, 4), 256, 0, st>>>(                                             \
        part, cnt, nullptr, 1, q0, mx, S, nq, kp, k, Xq, X.ld, X.data, X.ld, X.d, zn + q0, mx, err_coef, ed, 2.0f * ea, 1, n - 1, \
        KNN_OUT_SQL2, Hn + q0 * k, Hd + q0 * k, fb_rows, (int*)fb_count);                                            \
    exact_fallback_kernel<DT><<<1024, 256, 0, st>>>(fb_rows, (int*)fb_count, Xq, X.ld, X.data, X.ld, n, X.d, nullptr, \
                                                    1, q0, k, KNN_OUT_SQL2, Hn + q0 * k, Hd + q0 * k, part, nq * S,  \
                                                    fb_count + 1)
            if (X.dtype == KNN_F32) {
                KNN_QMR(KNN_F32);
            } else if (X.dtype == KNN_BF16) {
                KNN_QMR(KNN_BF16);
            } else {
                KNN_QMR(KNN_F16);
            }
#undef KNN_QMR
            KNN_HIP(hipGetLastError());
        }
        return KNN_OK;
    };
    auto rank_direct = [&](const float* Zs, int ldz, int dz, const uint64_t* pz, uint32_t* cz) {
        // reference splits (counts added) so that enough waves hide the tile reads
        const int64_t nb = ceil_div(n, 256);
        int Sd = (int)std::min<int64_t>(16, std::max<int64_t>(1, ceil_div(2048, nb)));
        Sd = (int)std::min<int64_t>(Sd, ceil_div(n, 256));
        const int64_t sl = round_up(ceil_div(n, Sd), 256);
        Sd = (int)ceil_div(n, sl);
        zero_words_kernel<<<(unsigned)std::min<int64_t>(ceil_div(n * kRankP, 64), 4096), 64, 0, st>>>(cz,
                                                                                                 n * kRankP);
        const dim3 g((unsigned)nb, (unsigned)Sd);
#define KNN_RD(DC)                                                                          \
    if (k <= 8) rank_direct_kernel<DC, 8><<<g, 256, 0, st>>>(Zs, n, ldz, dz, pz, sl, cz);          \
    else if (k <= 12) rank_direct_kernel<DC, 12><<<g, 256, 0, st>>>(Zs, n, ldz, dz, pz, sl, cz);   \
    else rank_direct_kernel<DC, 16><<<g, 256, 0, st>>>(Zs, n, ldz, dz, pz, sl, cz)
        if (dz == 2) {
            KNN_RD(2);
        } else if (dz == 3) {
            KNN_RD(3);
        } else {
            KNN_RD(0);
        }
#undef KNN_RD
    };
    if (!fused) {
        rank_direct((const float*)Xs, ldx, X.d, pu, cu);
    } else {
        if ((r = rank_tile((const float*)Xs, xn, ldx, X.d, pu, small, cu, true)) != KNN_OK) return r;
        quality_probes_kernel<<<(unsigned)ceil_div(n, 4), 256, 0, st>>>(n, k, Hn, Ln, (const float*)Xs, ldx, X.d,
                                                                        (const float*)Ys, ldy, Y.d, nullptr, pv,
                                                                        hits, 0);
    }
    if (Y.d <= kRankDirectD)
        rank_direct((const float*)Ys, ldy, Y.d, pv, cv);
    else if ((r = rank_tile((const float*)Ys, yn, ldy, Y.d, pv, small + 1, cv, false)) != KNN_OK)
        return r;
    KNN_HIP(hipGetLastError());
    unsigned long long* tot = (unsigned long long*)(small + 2);
    quality_reduce_kernel<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(n, k, pu, cu, pv, cv, hits, trust_out,
                                                                      cont_out, tot);
    KNN_HIP(hipGetLastError());
    unsigned long long host[3];
    KNN_HIP(hipMemcpyAsync(host, tot, 24, hipMemcpyDeviceToHost, st));
    KNN_HIP(hipStreamSynchronize(st));
    const double nk = (double)n * (double)k;
    const double z = 2.0 / (nk * (2.0 * (double)n - 3.0 * (double)k - 1.0));
    metrics[0] = (double)host[0] / nk;
    metrics[1] = 1.0 - z * (double)host[1];
    metrics[2] = 1.0 - z * (double)host[2];
    return KNN_OK;
}

// ------------------------------------------------------------ no-alloc path

// The static scratch array of knn_exact_noalloc: one copy per device, held
// by the loaded code object until the process ends.  Host code never uses
// this name as an address (on the host it is a stand-in symbol): the device
// address comes from hipGetSymbolAddress, once per device.
constexpr size_t kStaticScratch = (size_t)KNN_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratch];

static knn_status static_scratch(void** out)
{
    static std::mutex mu;
    static void* addr[64] = {};
    int dev = -1;
    KNN_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return fail(KNN_EDEVICE, "device ordinal out of range");
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(KNN_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        addr[dev] = p;
    }
    *out = addr[dev];
    return KNN_OK;
}

}  // namespace knn

using namespace knn;

extern "C" knn_status knn_exact(knn_matrix X, int32_t k, int32_t precision, int32_t rerank_k,
                                int32_t out_kind, int32_t* out_idx, float* out_dist, void* stream)
{
    try {
        knn_status r = check_matrix(X, "X");
        if (r != KNN_OK) return r;
        if (X.n < 2) return fail(KNN_EINVAL, "X.n must be >= 2");
        hipStream_t st = (hipStream_t)stream;
        Workspace ws(st, 0);
        return exact_impl(X, X, true, nullptr, 1, k, precision, rerank_k, out_kind, out_idx,
                          out_dist, st, ws, 0);
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}

extern "C" knn_status knn_exact_query(knn_matrix Q, knn_matrix R, const int32_t* q_self,
                                      int32_t k, int32_t precision, int32_t rerank_k,
                                      int32_t out_kind, int32_t* out_idx, float* out_dist,
                                      void* stream)
{
    try {
        knn_status r = check_matrix(Q, "Q");
        if (r != KNN_OK) return r;
        r = check_matrix(R, "R");
        if (r != KNN_OK) return r;
        if (Q.d != R.d) return fail(KNN_EINVAL, "Q.d != R.d");
        if (Q.dtype != R.dtype) return fail(KNN_EINVAL, "Q.dtype != R.dtype");
        hipStream_t st = (hipStream_t)stream;
        Workspace ws(st, 0);
        return exact_impl(Q, R, false, q_self, q_self ? 2 : 0, k, precision, rerank_k, out_kind,
                          out_idx, out_dist, st, ws, 0);
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}

extern "C" knn_status knn_exact_query_limited(knn_matrix Q, knn_matrix R, const int32_t* q_self,
                                              int32_t k, int32_t precision, int32_t rerank_k,
                                              int32_t out_kind, int64_t workspace_limit_bytes,
                                              int32_t* out_idx, float* out_dist, void* stream)
{
    try {
        knn_status r = check_matrix(Q, "Q");
        if (r != KNN_OK) return r;
        r = check_matrix(R, "R");
        if (r != KNN_OK) return r;
        if (Q.d != R.d) return fail(KNN_EINVAL, "Q.d != R.d");
        if (Q.dtype != R.dtype) return fail(KNN_EINVAL, "Q.dtype != R.dtype");
        hipStream_t st = (hipStream_t)stream;
        Workspace ws(st, 0);
        return exact_impl(Q, R, false, q_self, q_self ? 2 : 0, k, precision, rerank_k, out_kind,
                          out_idx, out_dist, st, ws, workspace_limit_bytes);
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}

extern "C" knn_status knn_exact_noalloc(knn_matrix X, int32_t k, int32_t precision, int32_t rerank_k,
                                        int32_t out_kind, int32_t* out_idx, float* out_dist, void* stream)
{
    try {
        knn_status r = check_matrix(X, "X");
        if (r != KNN_OK) return r;
        if (X.n < 2) return fail(KNN_EINVAL, "X.n must be >= 2");
        void* base = nullptr;
        if ((r = static_scratch(&base)) != KNN_OK) return r;
        FixedScratch ws(base, kStaticScratch);
        return exact_impl(X, X, true, nullptr, 1, k, precision, rerank_k, out_kind, out_idx,
                          out_dist, (hipStream_t)stream, ws, (int64_t)kStaticScratch);
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}

extern "C" knn_status knn_quality(knn_matrix X, knn_matrix Y, int32_t k, int32_t* hits, int64_t* trust,
                                  int64_t* cont, double* metrics, void* stream)
{
    try {
        knn_status r = check_matrix(X, "X");
        if (r != KNN_OK) return r;
        if ((r = check_matrix(Y, "Y")) != KNN_OK) return r;
        if (!metrics) return fail(KNN_EINVAL, "metrics is null");
        if (X.n != Y.n) return fail(KNN_EINVAL, "X.n != Y.n");
        if (k < 1 || 3 * (int64_t)k >= 2 * X.n - 1) return fail(KNN_EINVAL, "k must satisfy 1 <= k and 3k < 2n - 1");
        if (k > kRankP) return fail(KNN_ENOTSUP, "k above 16 is not supported by the quality metrics");
        return quality_impl(X, Y, k, hits, trust, cont, metrics, (hipStream_t)stream);
    } catch (...) {
        return fail(KNN_EDEVICE, "unexpected exception");
    }
}
