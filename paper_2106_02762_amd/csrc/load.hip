// Loading a temporal graph: the static graph G and the per-pair, per-direction edge store
// (Section 3 defines G and the multiplicities; Section 4 assumes constant-time access to each
// pair's edges in each direction in time order, which this CSR store provides).
//
// Every kept edge gets the 64-bit key ((t - t_min) << shift) | input_index, so that one unsigned
// comparison orders edges by (t, input index) and a time bound "t < x" is the key bound
// (x - t_min) << shift.
//
// Bound by the radix passes of the pair sort (12 bytes an edge read and written in each) and the one
// random read per edge after it.  Inputs are usually logs in time order: their keys need no sort, a
// pair key holds no more bits than two ids do (a word while they fit), and the neighbour lists take
// a sort of the pairs' larger ends only.  Load plus one-shot count of 61M edges in time order:
// 53.7 ms with three 64-bit sorts, 36.7 ms so; load, build and count of 10M: 6.8 and 4.6 ms.
#include <algorithm>
#include <cstring>

#include "internal.h"

namespace dt {

namespace {

constexpr unsigned kBlock = 256;
constexpr unsigned kScanGrid = 512;   // blocks of the input scan (each leaves one row of partials)
constexpr unsigned kWaveTile = 1024;  // edges in pair order one wavefront takes

__device__ inline uint64_t order_key(int64_t t) {   // int64 -> uint64, order preserving
    return (uint64_t)t ^ 0x8000000000000000ull;
}

// One row per block: [0] bad ids, [1] self loops, [2] smallest and [3] largest time of the kept
// edges (as order keys), [4] places where a time is below the one before it.  The host adds the
// rows: thousands of blocks meeting at four counters cost more than the read itself on small inputs.
__global__ void k_scan_input(uint32_t n, uint64_t m, const uint32_t *__restrict__ src,
                             const uint32_t *__restrict__ dst, const int64_t *__restrict__ t,
                             unsigned long long *__restrict__ out) {
    __shared__ unsigned long long s_p[kBlock / 64][5];
    unsigned long long p[5] = {0, 0, ~0ull, 0, 0};
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < m;
         i += (uint64_t)gridDim.x * kBlock) {
        const uint32_t a = src[i], b = dst[i];
        const int64_t ti = t[i];
        if (i && ti < t[i - 1]) p[4]++;
        if (a >= n || b >= n) { p[0]++; continue; }
        if (a == b) { p[1]++; continue; }
        const uint64_t k = order_key(ti);
        p[2] = k < p[2] ? k : p[2];
        p[3] = k > p[3] ? k : p[3];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long mn = __shfl_xor(p[2], o, 64), mx = __shfl_xor(p[3], o, 64);
        p[0] += __shfl_xor(p[0], o, 64);
        p[1] += __shfl_xor(p[1], o, 64);
        p[2] = mn < p[2] ? mn : p[2];
        p[3] = mx > p[3] ? mx : p[3];
        p[4] += __shfl_xor(p[4], o, 64);
    }
    if ((threadIdx.x & 63) == 0)
        for (int x = 0; x < 5; ++x) s_p[threadIdx.x / 64][x] = p[x];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned w = 1; w < kBlock / 64; ++w) {
            p[0] += s_p[w][0];
            p[1] += s_p[w][1];
            p[2] = s_p[w][2] < p[2] ? s_p[w][2] : p[2];
            p[3] = s_p[w][3] > p[3] ? s_p[w][3] : p[3];
            p[4] += s_p[w][4];
        }
        for (int x = 0; x < 5; ++x) out[5 * blockIdx.x + x] = p[x];
    }
}

// time key of every input edge; self-loops get ~0 so that they sort last
__global__ void k_time_keys(uint64_t m, const uint32_t *__restrict__ src,
                            const uint32_t *__restrict__ dst, const int64_t *__restrict__ t,
                            int64_t t_min, int shift, uint64_t *__restrict__ key,
                            uint32_t *__restrict__ idx) {
    uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= m) return;
    key[i] = src[i] == dst[i] ? ~0ull : ((uint64_t)(t[i] - t_min) << shift) | i;
    idx[i] = (uint32_t)i;
}

// Unordered pair (x << nb | y, x < y, 2^nb >= n) of each edge in time order, with its place in that
// order and its direction (1: y -> x) in the top bit.  idx_t: input index of each place (null: the
// input is in time order itself).  Self-loops (only with idx_t null) get a key past every pair's.
template <class K>
__global__ void k_pair_keys(uint64_t m, const uint32_t *__restrict__ idx_t, const uint32_t *__restrict__ src,
                            const uint32_t *__restrict__ dst, int nb, K *__restrict__ pk,
                            uint32_t *__restrict__ jd) {
    const uint64_t j = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= m) return;
    const uint64_t i = idx_t ? idx_t[j] : j;
    const uint32_t a = src[i], b = dst[i];
    const uint32_t x = a < b ? a : b, y = a < b ? b : a;
    const K top = ((K)1 << nb) - 1;
    pk[j] = a == b ? (K)(top << nb | top) : (K)((K)x << nb | y);
    jd[j] = (uint32_t)j | (a > b ? 0x80000000u : 0u);
}

// per wavefront tile of the edges in pair order: pairs that begin there (high word) and edges
// y -> x (low word)
template <class K>
__global__ void k_pair_count(uint64_t m, uint64_t tiles, const K *__restrict__ pk, const uint32_t *__restrict__ jd,
                             uint64_t *__restrict__ cnt) {
    const uint64_t tile = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / 64;
    const unsigned lane = threadIdx.x & 63;
    if (tile > tiles) return;
    uint32_t heads = 0, back = 0;
#pragma unroll 4
    for (unsigned r = 0; r < kWaveTile / 64; ++r) {
        const uint64_t k = tile * kWaveTile + r * 64 + lane;
        const bool in = k < m;
        const K p = in ? pk[k] : 0, q = in && k ? pk[k - 1] : 0;
        heads += (uint32_t)__popcll(__ballot(in && (k == 0 || p != q)));
        back += (uint32_t)__popcll(__ballot(in && (jd[in ? k : 0] >> 31) != 0));
    }
    if (lane == 0) cnt[tile] = tile < tiles ? (uint64_t)heads << 32 | back : 0;
}

// Per edge in pair order: pair id, key, direction and the edges y -> x before it; per pair: its
// endpoints and first edge.  base: the exclusive scan of k_pair_count.  Keys come from tkey (by
// place in time order) or, when the input is in time order, from the times themselves.  One random
// read per edge (its key or time); the rest streams.
template <class K>
__global__ void k_fill_pairs(uint64_t m, uint64_t tiles, const K *__restrict__ pk, const uint32_t *__restrict__ jd,
                             const uint64_t *__restrict__ base, const uint64_t *__restrict__ tkey,
                             const int64_t *__restrict__ t, int64_t t_min, int shift, int nb,
                             uint32_t *__restrict__ psid, uint64_t *__restrict__ pkey, uint8_t *__restrict__ pdir,
                             uint32_t *__restrict__ sx, uint32_t *__restrict__ sy, uint32_t *__restrict__ pstart,
                             uint32_t *__restrict__ c1) {
    const uint64_t tile = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / 64;
    const unsigned lane = threadIdx.x & 63;
    if (tile >= tiles) return;
    uint32_t s0 = (uint32_t)(base[tile] >> 32), b0 = (uint32_t)base[tile];
    const uint64_t below = (1ull << lane) - 1;
#pragma unroll 4
    for (unsigned r = 0; r < kWaveTile / 64; ++r) {
        const uint64_t k = tile * kWaveTile + r * 64 + lane;
        const bool in = k < m;
        const K p = in ? pk[k] : 0, q = in && k ? pk[k - 1] : 0;
        const uint32_t v = in ? jd[k] : 0, j = v & 0x7fffffffu;
        const bool head = in && (k == 0 || p != q), back = (v >> 31) != 0;
        const uint64_t hm = __ballot(head), bm = __ballot(back);
        if (in) {
            const uint32_t s = s0 + (uint32_t)__popcll(hm & below) - (head ? 0u : 1u);
            psid[k] = s;
            pkey[k] = tkey ? tkey[j] : ((uint64_t)(t[j] - t_min) << shift) | j;
            pdir[k] = back ? 1 : 0;
            c1[k] = b0 + (uint32_t)__popcll(bm & below);
            if (head) {
                sx[s] = (uint32_t)(p >> nb);
                sy[s] = (uint32_t)(p & (((K)1 << nb) - 1));
                pstart[s] = (uint32_t)k;
            }
            if (k == m - 1) {
                c1[m] = b0 + (uint32_t)__popcll(bm);
                pstart[s + 1] = (uint32_t)m;
            }
        }
        s0 += (uint32_t)__popcll(hm);
        b0 += (uint32_t)__popcll(bm);
    }
}

__device__ __forceinline__ uint32_t first_at_least(const uint32_t *__restrict__ a, uint64_t len, uint32_t x) {
    uint64_t lo = 0;
    while (len > 0) {
        const uint64_t half = len >> 1;
        if (a[lo + half] < x) {
            lo += half + 1;
            len -= half + 1;
        } else {
            len = half;
        }
    }
    return (uint32_t)lo;
}

// Rows of the undirected CSR: v's smaller neighbours are the pairs (x, v) (ys: the pairs' larger
// ends, sorted), its larger ones the pairs (v, y) (sx, sorted already).  xrow[v]: pairs with a
// smaller first end than v.
__global__ void k_rows(uint32_t n, uint64_t ms, const uint32_t *__restrict__ sx, const uint32_t *__restrict__ ys,
                       uint32_t *__restrict__ xrow, uint32_t *__restrict__ row) {
    const uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (v > n) return;
    const uint32_t a = first_at_least(sx, ms, (uint32_t)v), b = first_at_least(ys, ms, (uint32_t)v);
    xrow[v] = a;
    row[v] = a + b;
}

// Neighbours in their rows, by id: entry q of the pairs by larger end goes after the larger
// neighbours of every earlier vertex, pair s after the smaller neighbours of every vertex up to its
// own.  Also the most edges on one pair.
__global__ void k_cols(uint64_t ms, const uint32_t *__restrict__ sx, const uint32_t *__restrict__ sy,
                       const uint32_t *__restrict__ ys, const uint32_t *__restrict__ xs,
                       const uint32_t *__restrict__ xrow, const uint32_t *__restrict__ row,
                       const uint32_t *__restrict__ pstart, uint32_t *__restrict__ col, unsigned *__restrict__ max_mult) {
    unsigned mx = 0;
    for (uint64_t s = (uint64_t)blockIdx.x * kBlock + threadIdx.x; s < ms; s += (uint64_t)gridDim.x * kBlock) {
        const uint32_t x = sx[s], y = ys[s];
        col[s + row[x + 1] - xrow[x + 1]] = sy[s];
        col[s + xrow[y]] = xs[s];
        const unsigned c = pstart[s + 1] - pstart[s];
        mx = c > mx ? c : mx;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned y = __shfl_xor(mx, o, 64);
        mx = y > mx ? y : mx;
    }
    __shared__ unsigned s_mx[kBlock / 64];
    if ((threadIdx.x & 63) == 0) s_mx[threadIdx.x / 64] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned w = 1; w < kBlock / 64; ++w) mx = s_mx[w] > mx ? s_mx[w] : mx;
        atomicMax(max_mult, mx);
    }
}

int bits_for(uint64_t x) {   // smallest b >= 1 with x <= 2^b
    int b = 1;
    while (b < 64 && (1ull << b) < x) b++;
    return b;
}

// The pair-major store from the edges in time order (tkey and idx_t; both null when the input is in
// time order, whose self-loops then sort last here): pair keys of K, nb bits per end.
template <class K>
int group_pairs(dt_graph *g, const uint32_t *src, const uint32_t *dst, const int64_t *t, const uint64_t *tkey,
                const uint32_t *idx_t, int nb, unsigned *max_mult) {
    dt_ctx *ctx = g->ctx;
    hipStream_t st = ctx->stream;
    const uint64_t m = g->m, m_sort = idx_t ? m : g->m_in;
    DevMem pk, pk2, jd, jd2, cnt, base;
    DT_TRY(dev_alloc(ctx, pk, m_sort * sizeof(K)));
    DT_TRY(dev_alloc(ctx, jd, m_sort * 4));
    DT_TRY(dev_alloc(ctx, pk2, m_sort * sizeof(K)));
    DT_TRY(dev_alloc(ctx, jd2, m_sort * 4));
    k_pair_keys<K><<<grid_for(m_sort, kBlock), kBlock, 0, st>>>(m_sort, idx_t, src, dst, nb, pk.as<K>(),
                                                                jd.as<uint32_t>());
    DT_HIP(hipGetLastError());
    // stable, so each pair's edges stay in key order
    if constexpr (sizeof(K) == 4)
        DT_TRY(sort_pairs_u32_u32(ctx, pk.as<uint32_t>(), pk2.as<uint32_t>(), jd.as<uint32_t>(), jd2.as<uint32_t>(),
                                  m_sort, 2 * nb, st));
    else
        DT_TRY(sort_pairs_u64_u32(ctx, pk.as<uint64_t>(), pk2.as<uint64_t>(), jd.as<uint32_t>(), jd2.as<uint32_t>(),
                                  m_sort, 2 * nb, st));
    pk.reset();
    jd.reset();
    const uint64_t tiles = (m + kWaveTile - 1) / kWaveTile;
    DT_TRY(dev_alloc(ctx, cnt, (tiles + 1) * 8));
    DT_TRY(dev_alloc(ctx, base, (tiles + 1) * 8));
    k_pair_count<K><<<grid_for(tiles + 1, kBlock / 64), kBlock, 0, st>>>(m, tiles, pk2.as<K>(), jd2.as<uint32_t>(),
                                                                         cnt.as<uint64_t>());
    DT_HIP(hipGetLastError());
    DT_TRY(exclusive_scan_u64(ctx, cnt.as<uint64_t>(), base.as<uint64_t>(), tiles + 1, st));
    uint64_t *h = reinterpret_cast<uint64_t *>(ctx->pinned_stage);
    DT_HIP(hipMemcpyAsync(h, base.as<uint64_t>() + tiles, 8, hipMemcpyDeviceToHost, st));
    DT_HIP(hipStreamSynchronize(st));
    const uint64_t ms = h[0] >> 32;
    g->m_s = ms;
    DT_TRY(dev_alloc(ctx, g->sx, ms * 4));
    DT_TRY(dev_alloc(ctx, g->sy, ms * 4));
    DT_TRY(dev_alloc(ctx, g->pstart, (ms + 1) * 4));
    DT_TRY(dev_alloc(ctx, g->psid, m * 4));
    DT_TRY(dev_alloc(ctx, g->pkey, m * 8));
    DT_TRY(dev_alloc(ctx, g->pdir, m));
    DT_TRY(dev_alloc(ctx, g->c1, (m + 1) * 4));
    k_fill_pairs<K><<<grid_for(tiles, kBlock / 64), kBlock, 0, st>>>(
        m, tiles, pk2.as<K>(), jd2.as<uint32_t>(), base.as<uint64_t>(), tkey, t, g->t_min, g->shift, nb,
        g->psid.as<uint32_t>(), g->pkey.as<uint64_t>(), g->pdir.as<uint8_t>(), g->sx.as<uint32_t>(),
        g->sy.as<uint32_t>(), g->pstart.as<uint32_t>(), g->c1.as<uint32_t>());
    DT_HIP(hipGetLastError());
    pk2.reset();
    jd2.reset();
    // undirected CSR of G, neighbours by id: the pairs are sorted by their smaller end, so only the
    // larger ends are left to sort
    DevMem ys, xs, xrow;
    DT_TRY(dev_alloc(ctx, ys, ms * 4));
    DT_TRY(dev_alloc(ctx, xs, ms * 4));
    DT_TRY(dev_alloc(ctx, xrow, ((uint64_t)g->n + 1) * 4));
    DT_TRY(dev_alloc(ctx, g->row, ((uint64_t)g->n + 1) * 4));
    DT_TRY(dev_alloc(ctx, g->col, 2 * ms * 4));
    DT_TRY(sort_pairs_u32_u32(ctx, g->sy.as<uint32_t>(), ys.as<uint32_t>(), g->sx.as<uint32_t>(), xs.as<uint32_t>(), ms,
                              nb, st));
    k_rows<<<grid_for((uint64_t)g->n + 1, kBlock), kBlock, 0, st>>>(g->n, ms, g->sx.as<uint32_t>(), ys.as<uint32_t>(),
                                                                    xrow.as<uint32_t>(), g->row.as<uint32_t>());
    DT_HIP(hipGetLastError());
    const unsigned grid = std::min<unsigned>(grid_for(ms, kBlock), (unsigned)ctx->num_cus * 8);
    k_cols<<<grid, kBlock, 0, st>>>(ms, g->sx.as<uint32_t>(), g->sy.as<uint32_t>(), ys.as<uint32_t>(), xs.as<uint32_t>(),
                                    xrow.as<uint32_t>(), g->row.as<uint32_t>(), g->pstart.as<uint32_t>(),
                                    g->col.as<uint32_t>(), max_mult);
    DT_HIP(hipGetLastError());
    return DT_OK;
}

}  // namespace

int load_graph(dt_graph *g, const uint32_t *src, const uint32_t *dst, const int64_t *t) {
    dt_ctx *ctx = g->ctx;
    hipStream_t st = ctx->stream;
    const uint64_t m_in = g->m_in;
    const uint32_t n = g->n;

    // 1. validate ids, count self-loops, time range, and whether the input is in time order
    DevMem scal;
    static_assert(kScanGrid * 5 * 8 <= kPinnedStage, "staging layout");
    DT_TRY(dev_alloc(ctx, scal, kScanGrid * 5 * 8));
    uint64_t h[5] = {0, 0, ~0ull, 0, 0};
    if (m_in) {
        const unsigned grid = std::min(grid_for(m_in, kBlock), kScanGrid);
        k_scan_input<<<grid, kBlock, 0, st>>>(n, m_in, src, dst, t, scal.as<unsigned long long>());
        DT_HIP(hipGetLastError());
        uint64_t *p = reinterpret_cast<uint64_t *>(ctx->pinned_stage);
        DT_HIP(hipMemcpyAsync(p, scal.ptr, grid * 5 * 8, hipMemcpyDeviceToHost, st));
        DT_HIP(hipStreamSynchronize(st));
        for (unsigned b = 0; b < grid; ++b) {
            h[0] += p[5 * b];
            h[1] += p[5 * b + 1];
            h[2] = std::min(h[2], p[5 * b + 2]);
            h[3] = std::max(h[3], p[5 * b + 3]);
            h[4] += p[5 * b + 4];
        }
    }
    if (h[0]) return fail(DT_EINVAL, "%llu edges name a vertex id >= n = %u", (unsigned long long)h[0], n);
    g->self_loops = h[1];
    g->m = m_in - h[1];
    const uint64_t m = g->m;
    if (m) {
        g->t_min = (int64_t)(h[2] ^ 0x8000000000000000ull);
        g->t_max = (int64_t)(h[3] ^ 0x8000000000000000ull);
    } else {
        g->t_min = g->t_max = 0;
    }
    g->span = g->t_max - g->t_min;
    g->shift = bits_for(m_in);
    if (m && ((uint64_t)g->span >> (64 - g->shift)) != 0)
        return fail(DT_EOVERFLOW, "time span %lld does not fit beside a %d-bit edge index",
                    (long long)g->span, g->shift);
    if (m && (uint64_t)g->span + 2 >= (1ull << (64 - g->shift)))
        return fail(DT_EOVERFLOW, "time span %lld too close to the %d-bit key limit",
                    (long long)g->span, 64 - g->shift);
    g->max_mult = 0;
    g->m_s = 0;
    if (m == 0) {
        for (DevMem *a : {&g->sx, &g->sy, &g->psid, &g->pkey, &g->pdir, &g->col}) DT_TRY(dev_alloc(ctx, *a, 0));
        DT_TRY(dev_alloc(ctx, g->pstart, 4));
        DT_TRY(dev_alloc(ctx, g->c1, 4));
        DT_TRY(dev_alloc(ctx, g->row, ((uint64_t)n + 1) * 4));
        DT_HIP(hipMemsetAsync(g->pstart.ptr, 0, 4, st));
        DT_HIP(hipMemsetAsync(g->c1.ptr, 0, 4, st));
        DT_HIP(hipMemsetAsync(g->row.ptr, 0, ((uint64_t)n + 1) * 4, st));
        DT_HIP(hipStreamSynchronize(st));
        return DT_OK;
    }

    // 2. keys in (t, index) order: the input's own order when its times never decrease (as the
    // inputs of Section 5 are), else sorted
    const bool sorted = h[4] == 0;
    DevMem tk2, tidx2;
    if (!sorted) {
        DevMem tk, tidx;
        DT_TRY(dev_alloc(ctx, tk, m_in * 8));
        DT_TRY(dev_alloc(ctx, tidx, m_in * 4));
        DT_TRY(dev_alloc(ctx, tk2, m_in * 8));
        DT_TRY(dev_alloc(ctx, tidx2, m_in * 4));
        k_time_keys<<<grid_for(m_in, kBlock), kBlock, 0, st>>>(m_in, src, dst, t, g->t_min, g->shift,
                                                               tk.as<uint64_t>(), tidx.as<uint32_t>());
        DT_HIP(hipGetLastError());
        DT_TRY(sort_pairs_u64_u32(ctx, tk.as<uint64_t>(), tk2.as<uint64_t>(), tidx.as<uint32_t>(),
                                  tidx2.as<uint32_t>(), m_in, 64, st));
    }

    // 3. grouped by unordered pair; pair keys of 32 bits while two ids fit them
    unsigned *mm = scal.as<unsigned>();
    DT_HIP(hipMemsetAsync(mm, 0, 4, st));
    const int nb = bits_for(n);
    const uint64_t *tkey = sorted ? nullptr : tk2.as<uint64_t>();
    const uint32_t *idx_t = sorted ? nullptr : tidx2.as<uint32_t>();
    DT_TRY(2 * nb <= 32 ? group_pairs<uint32_t>(g, src, dst, t, tkey, idx_t, nb, mm)
                        : group_pairs<uint64_t>(g, src, dst, t, tkey, idx_t, nb, mm));
    DT_HIP(hipMemcpyAsync(ctx->pinned_stage, mm, 4, hipMemcpyDeviceToHost, st));
    DT_HIP(hipStreamSynchronize(st));
    memcpy(&g->max_mult, ctx->pinned_stage, 4);
    return DT_OK;
}

}  // namespace dt
