// Exact k-NN of rows of one to three coordinates (e.g. a 2-D embedding) by
// direct canonical FP32 distances, pruned by boxes.
//
// The references are ordered along a space-filling curve (a Hilbert curve in
// two dimensions, Z-order in three) over a grid whose cells hold about equally
// many references per coordinate, and cut into tiles of 64 consecutive
// references and groups of 64 tiles, each with its bounding box.  A wave takes
// a query: starting from the query's own tile (or the one nearest to it) it visits the groups, and in
// them the tiles, whose box is not further than the current k-th distance,
// one reference per lane, and keeps the 64 smallest keys (canonical distance,
// index) sorted across its lanes.  A tile that is skipped cannot hold a
// neighbour (see box_d2), and keys are totally ordered, so the result is that
// of a search over all pairs.
//
// Over all pairs the 70,000 x 2 search (k = 10) is 4.9e9 distances and gates, VALU
// work of 2.49 ms; it takes 0.14 ms here, 0.11 of them the search (a wave visits
// a few tiles; bound by VALU work of the list), the rest the sort.  From 4
// coordinates on boxes no longer prune, a tile's neighbourhood is most of the
// set (70,000 x 8: 12 ms here, 7.3 over all pairs).
#include <algorithm>

#include "knn_common.hpp"

namespace knn {

constexpr int kLdTile = 64;      // references per tile, tiles per group
constexpr int kLdCells = 256;    // cells per coordinate
constexpr int kLdSample = 1024;  // references sampled for their boundaries

// One workgroup per coordinate t: bnd[t][c], the lower boundary of cell c (c >
// 0), and the least and the largest sampled value at bnd[t][0] and
// bnd[t][kLdCells]; from kLdSample references at equal steps.
template <int DT>
__global__ __launch_bounds__(kLdSample) void ld_cells_kernel(const void* __restrict__ X, int64_t ld, int64_t n,
                                                             float* __restrict__ bnd)
{
    __shared__ uint32_t v[kLdSample];
    const int i = threadIdx.x, t = blockIdx.x;
    const uint32_t u = __float_as_uint(elem<DT>::ld(X, (int64_t)i * n / kLdSample * ld + t));
    v[i] = u & 0x80000000u ? ~u : u | 0x80000000u;   // in the order of the values
    for (int w = 2; w <= kLdSample; w <<= 1) {
        for (int j = w >> 1; j > 0; j >>= 1) {
            __syncthreads();
            const int o = i ^ j;
            if (o > i) {
                const uint32_t a = v[i], b = v[o];
                if ((a > b) == ((i & w) == 0)) {
                    v[i] = b;
                    v[o] = a;
                }
            }
        }
    }
    __syncthreads();
    if (i <= kLdCells) {
        const uint32_t s = v[i < kLdCells ? i * (kLdSample / kLdCells) : kLdSample - 1];
        bnd[t * (kLdCells + 1) + i] = __uint_as_float(s & 0x80000000u ? s & 0x7FFFFFFFu : ~s);
    }
}

// Position of cell (x, y) on the Hilbert curve over 2^bits x 2^bits cells, by the
// curve's recursive definition (Hilbert 1891): one quadrant per level, the lower
// quadrants' curves transposed (and mirrored).
__device__ inline uint32_t hilbert(uint32_t x, uint32_t y, int bits)
{
    uint32_t pos = 0;
    for (int b = bits - 1; b >= 0; --b) {
        const uint32_t qx = (x >> b) & 1u, qy = (y >> b) & 1u;
        pos = (pos << 2) | ((3u * qx) ^ qy);
        if (qy == 0u) {
            if (qx == 1u) {
                x = ~x;
                y = ~y;
            }
            const uint32_t t = x;
            x = y;
            y = t;
        }
    }
    return pos;
}

// Curve position of every row, `bits` bits per coordinate: its cell's, the low
// ones from its place between the cell's boundaries above 8 bits.
template <int DT>
__global__ __launch_bounds__(256) void ld_key_kernel(const void* __restrict__ X, int64_t ld, int64_t n, int d,
                                                     int bits, const float* __restrict__ bnd,
                                                     uint32_t* __restrict__ key, uint32_t* __restrict__ val)
{
    __shared__ float sb[kLowdimD][kLdCells + 1];
    for (int i = threadIdx.x; i < d * (kLdCells + 1); i += 256) sb[i / (kLdCells + 1)][i % (kLdCells + 1)] = bnd[i];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    uint32_t c[kLowdimD] = {0u, 0u, 0u};
#pragma unroll
    for (int t = 0; t < kLowdimD; ++t) {
        if (t >= d) continue;
        const float x = elem<DT>::ld(X, i * ld + t);
        uint32_t m = 0;   // boundaries not above x, of those from cell 1 on
#pragma unroll
        for (uint32_t h = kLdCells / 2; h > 0; h >>= 1) m += sb[t][m + h] <= x ? h : 0u;
        if (bits <= 8) {
            c[t] = m >> (8 - bits);
        } else {
            const float lo = sb[t][m], hi = sb[t][m + 1], cells = (float)(1 << (bits - 8));
            const float f = hi > lo ? (x - lo) / (hi - lo) * cells : 0.0f;
            c[t] = (m << (bits - 8)) | (f > 0.0f ? (f < cells ? (uint32_t)f : (uint32_t)cells - 1u) : 0u);
        }
    }
    uint32_t k = c[0];
    if (d == 2) k = hilbert(c[0], c[1], bits);
    if (d == 3) {
        k = 0;
        for (int b = bits - 1; b >= 0; --b)
            k = (k << 3) | (((c[0] >> b) & 1u) << 2) | (((c[1] >> b) & 1u) << 1) | ((c[2] >> b) & 1u);
    }
    key[i] = k;
    val[i] = (uint32_t)i;
}

// One wave per tile: the tile's rows in curve order, coordinate t of position p
// at S[t * np + p] (FP32), its box (lowest at box[t * nt + tile], highest
// at box[(d + t) * nt + tile]) and its least row number.
template <int DT>
__global__ __launch_bounds__(256) void ld_tiles_kernel(const void* __restrict__ X, int64_t ld, int64_t n, int d,
                                                       const uint32_t* __restrict__ order, int64_t np, int64_t nt,
                                                       float* __restrict__ S, float* __restrict__ box,
                                                       uint32_t* __restrict__ low)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x, tile = p >> 6;
    if (tile >= nt) return;   // the whole wave
    const int64_t row = order[p < n ? p : n - 1];   // past the end: the last point again
    uint32_t lr = (uint32_t)row;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lr = min(lr, xor_u32(lr, o));
    if ((threadIdx.x & 63) == 0) low[tile] = lr;
    // a tile with an infinite or NaN coordinate gets the box of the whole
    // space: a distance to it may be NaN, which counts as 0
    bool finite = true;
    for (int t = 0; t < d; ++t) finite = finite && fabsf(elem<DT>::ld(X, row * ld + t)) < __builtin_inff();
    const bool whole = ballot(!finite) != 0;
    for (int t = 0; t < d; ++t) {
        const float x = elem<DT>::ld(X, row * ld + t);
        S[t * np + p] = x;
        float lo = x, hi = x;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fminf(lo, xor_f32(lo, o));
            hi = fmaxf(hi, xor_f32(hi, o));
        }
        if ((threadIdx.x & 63) == 0) {
            box[t * nt + tile] = whole ? -__builtin_inff() : lo;
            box[(d + t) * nt + tile] = whole ? __builtin_inff() : hi;
        }
    }
}

// One wave per group of 64 tiles: its box and least row number, as the tiles'.
__global__ __launch_bounds__(256) void ld_groups_kernel(const float* __restrict__ box, const uint32_t* __restrict__ low,
                                                        int64_t nt, int d, int64_t ng, float* __restrict__ gbox,
                                                        uint32_t* __restrict__ glow)
{
    const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= ng) return;
    const int64_t tile = g * kLdTile + (threadIdx.x & 63), b = tile < nt ? tile : nt - 1;
    uint32_t lr = low[b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) lr = min(lr, xor_u32(lr, o));
    if ((threadIdx.x & 63) == 0) glow[g] = lr;
    for (int t = 0; t < d; ++t) {
        float lo = box[t * nt + b], hi = box[(d + t) * nt + b];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fminf(lo, xor_f32(lo, o));
            hi = fmaxf(hi, xor_f32(hi, o));
        }
        if ((threadIdx.x & 63) == 0) {
            gbox[t * ng + g] = lo;
            gbox[(d + t) * ng + g] = hi;
        }
    }
}

// A wave's squared distances from its query to boxes base + lane (of nb), lower
// bounds of the canonical distances to what they hold: each gap is at most the
// coordinate's rounded difference, and the roundings of both sums (a few times
// 6e-8 relative, or 1e-45 among denormals) and an overflow are within the slack.  A
// query with an infinite or NaN coordinate is at distance 0 from
// every box.  +inf past the last box.
template <int D>
__device__ inline float box_d2(const float (&xq)[D], const float* __restrict__ box, int64_t nb, int64_t i)
{
    const int64_t b = i < nb ? i : nb - 1;
    float s = 0.0f;
    bool finite = true;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        const float g = fmaxf(box[t * nb + b] - xq[t], xq[t] - box[(D + t) * nb + b]);
        s = g > 0.0f ? fmaf(g, g, s) : s;
        finite = finite && fabsf(xq[t]) < __builtin_inff();
    }
    s = finite ? fminf(s, 3.402823466e38f) * 0.99999f - 1e-36f : -1.0f;
    return i < nb ? s : __builtin_inff();
}

// qorder: the queries in curve order (they are the references), or null.
template <int DT, int D>
__global__ __launch_bounds__(256) void ld_search_kernel(
    const void* __restrict__ Q, int64_t ldq, int64_t nq, const uint32_t* __restrict__ qorder,
    const float* __restrict__ S, const uint32_t* __restrict__ order, int64_t nr, int64_t np,
    const float* __restrict__ box, const uint32_t* __restrict__ low, int64_t nt, const float* __restrict__ gbox,
    const uint32_t* __restrict__ glow, int64_t ng,
    const int32_t* __restrict__ q_self, int self_mode, int k, int out_kind, int32_t* __restrict__ out_idx,
    float* __restrict__ out_dist)
{
    const int lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (p >= nq) return;
    const int64_t q = qorder ? (int64_t)__builtin_amdgcn_readfirstlane((int)qorder[p]) : p;
    const int64_t self = self_mode == 1 ? q : (self_mode == 2 ? (int64_t)q_self[q] : -1);
    float xq[D];
#pragma unroll
    for (int t = 0; t < D; ++t) xq[t] = elem<DT>::ld(Q, q * ldq + t);
    auto keys = [&](int64_t tile) {
        const int64_t i = tile * kLdTile + lane;
        float x[D];
#pragma unroll
        for (int t = 0; t < D; ++t) x[t] = S[t * np + i];
        const uint32_t id = i < nr ? order[i] : 0u;
        return i < nr && (int64_t)id != self ? make_key(direct_d2<D>(xq, x, D), id) : kEmptyCand;
    };
    // A box at distance v (a lower bound) may hold a key below the k-th one.
    // At a k-th distance of 0 (copies) only a smaller row number is.
    uint64_t list, kth;
    auto open = [&](float v, const uint32_t* rows, int64_t n, int64_t i) {
        bool o = i < n && v <= key_d2(kth);
        if (key_d2(kth) == 0.0f) o = o && rows[i < n ? i : n - 1] < key_idx(kth);
        return o;
    };
    auto visit = [&](int64_t tile) {
        const uint64_t key = keys(tile);
        uint64_t m = ballot(key < kth);
        if (popc64(m) > 24) {   // 6: 185 us, 16 or 28: 171 us (70,000 x 2)
            list = seg_merge_sorted<64>(list, seg_sort<64>(key));
        } else {
            for (; m; m &= m - 1) {
                // entries above the key move up one place, the first takes it
                const uint64_t y = bcast_u64(key, __builtin_ctzll(m)), up = shift_up_u64(list);
                list = umin64(list, umax64(up, y));
            }
        }
        kth = bcast_u64(list, k - 1);
    };
    // the lane of the least of v, the first of equal ones
    auto least = [&](float v) {
        float w = v;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) w = fminf(w, xor_f32(w, o));
        return (int)__builtin_ctzll(ballot(v == w));
    };
    int64_t first;
    if (qorder) {
        first = p / kLdTile;
    } else {
        float best = __builtin_inff();
        int64_t bg = 0;
        for (int64_t g = lane; g < round_up(ng, kLdTile); g += kLdTile) {
            const float v = box_d2<D>(xq, gbox, ng, g);
            if (v < best) {
                best = v;
                bg = g;
            }
        }
        bg = bcast_u32((uint32_t)bg, least(best));
        first = bg * kLdTile + least(box_d2<D>(xq, box, nt, bg * kLdTile + lane));
    }
    list = umin64(seg_sort<64>(keys(first)), kEmptyList);
    kth = bcast_u64(list, k - 1);
    auto scan = [&](int64_t g) {
        const int64_t i = g * kLdTile + lane;
        const float v = box_d2<D>(xq, box, nt, i);
        uint64_t m = ballot(i != first && open(v, low, nt, i));
        while (m) {
            const int l = __builtin_ctzll(m);
            visit(g * kLdTile + l);
            m &= (m - 1) & ballot(open(v, low, nt, i));
        }
    };
    const int64_t g0 = first / kLdTile;
    scan(g0);
    for (int64_t b = 0; b < ng; b += kLdTile) {
        const float v = box_d2<D>(xq, gbox, ng, b + lane);
        uint64_t m = ballot(b + lane != g0 && open(v, glow, ng, b + lane));
        while (m) {
            const int l = __builtin_ctzll(m);
            scan(b + l);
            m &= (m - 1) & ballot(open(v, glow, ng, b + lane));
        }
    }
    if (lane < k) {
        const float d2 = key_d2(list);
        out_idx[q * k + lane] = (int32_t)key_idx(list);
        out_dist[q * k + lane] = out_kind == KNN_OUT_L2 ? sqrtf(d2) : d2;
    }
}

namespace {

template <int DT>
knn_status lowdim_typed(const knn_matrix& Q, const knn_matrix& R, bool same, const int32_t* q_self, int self_mode,
                        int k, int out_kind, int32_t* out_idx, float* out_dist, hipStream_t st, ScratchAlloc& ws)
{
    const int64_t n = R.n, nt = ceil_div(n, kLdTile), np = nt * kLdTile, ng = ceil_div(nt, kLdTile);
    const int d = R.d;
    // 2^16 grid cells (two radix passes), about one reference each; 2^24 for
    // more references
    const int bits = (n <= (1 << 18) ? 16 : 24) / d;
    uint32_t *key, *val, *k1, *v1, *counts;
    float *bnd, *S, *box, *gbox;
    uint32_t *low, *glow;
    knn_status r;
    if ((r = ws.alloc(&bnd, (size_t)d * (kLdCells + 1))) != KNN_OK) return r;
    if ((r = ws.alloc(&key, (size_t)n)) != KNN_OK) return r;
    if ((r = ws.alloc(&val, (size_t)n)) != KNN_OK) return r;
    if ((r = ws.alloc(&k1, (size_t)n)) != KNN_OK) return r;
    if ((r = ws.alloc(&v1, (size_t)n)) != KNN_OK) return r;
    if ((r = ws.alloc(&counts, radix_counts_words(n))) != KNN_OK) return r;
    if ((r = ws.alloc(&S, (size_t)np * d)) != KNN_OK) return r;
    if ((r = ws.alloc(&box, (size_t)nt * 2 * d)) != KNN_OK) return r;
    if ((r = ws.alloc(&gbox, (size_t)ng * 2 * d)) != KNN_OK) return r;
    if ((r = ws.alloc(&low, (size_t)nt)) != KNN_OK) return r;
    if ((r = ws.alloc(&glow, (size_t)ng)) != KNN_OK) return r;
    ld_cells_kernel<DT><<<(unsigned)d, kLdSample, 0, st>>>(R.data, R.ld, n, bnd);
    ld_key_kernel<DT><<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(R.data, R.ld, n, d, bits, bnd, key, val);
    KNN_HIP(hipGetLastError());
    if ((r = radix_sort_bits(key, val, k1, v1, n, counts, st, d * bits, 1)) != KNN_OK) return r;
    ld_tiles_kernel<DT><<<(unsigned)ceil_div(np, 256), 256, 0, st>>>(R.data, R.ld, n, d, val, np, nt, S, box,
                                                                     low);
    ld_groups_kernel<<<(unsigned)ceil_div(ng, 4), 256, 0, st>>>(box, low, nt, d, ng, gbox, glow);
    const unsigned g = (unsigned)ceil_div(Q.n, 4);
    const uint32_t* qorder = same ? val : nullptr;
#define KNN_LD(D)                                                                                                  \
    ld_search_kernel<DT, D><<<g, 256, 0, st>>>(Q.data, Q.ld, Q.n, qorder, S, val, n, np, box, low, nt, gbox, glow, ng,     \
                                               q_self, self_mode, k, out_kind, out_idx, out_dist)
    if (d == 1) KNN_LD(1);
    else if (d == 2) KNN_LD(2);
    else KNN_LD(3);
#undef KNN_LD
    KNN_HIP(hipGetLastError());
    return KNN_OK;
}

}  // namespace

knn_status lowdim_knn(const knn_matrix& Q, const knn_matrix& R, bool same, const int32_t* q_self, int self_mode,
                      int k, int out_kind, int32_t* out_idx, float* out_dist, hipStream_t st, ScratchAlloc& ws)
{
    if (R.dtype == KNN_F32)
        return lowdim_typed<KNN_F32>(Q, R, same, q_self, self_mode, k, out_kind, out_idx, out_dist, st, ws);
    if (R.dtype == KNN_BF16)
        return lowdim_typed<KNN_BF16>(Q, R, same, q_self, self_mode, k, out_kind, out_idx, out_dist, st, ws);
    return lowdim_typed<KNN_F16>(Q, R, same, q_self, self_mode, k, out_kind, out_idx, out_dist, st, ws);
}

}  // namespace knn
