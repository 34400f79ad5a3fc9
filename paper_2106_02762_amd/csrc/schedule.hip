// Count schedule, built once per graph (it does not depend on the deltas, Section 6 "running time
// independent of time periods").  A triangle with one temporal edge per pair becomes a unit record
// (its ordering, orientation and type fixed here, Figures 3 and 4 with Table 2); a triangle with
// few (uv edge, uw edge) pairs goes to the light path (one lane).  Every other triangle is split
// between the medium path, whose work is the number of close pairs (growing with d13), and the
// prefix-count procedures of Algorithms 1-3 (work (sigma_uv + sigma_uw) log sigma, Theorem 1) by a
// cost model: its pair budget is the prefix procedures' cost over the medium path's cost per pair.
// A triangle whose P = sigma_uv sigma_uw pairs fit the budget is always medium; one whose outer
// edges alone exceed it is always heavy; for the others (contested) a wavefront finds the largest
// level l such that its pairs within D(l) = 2^(l-1) - 1 of each other fit, by binary search over
// the levels with exact close-pair counts.  Contested triangles are sorted by descending level, so
// that a whole-span query walks a prefix of the medium list and a suffix of the heavy list.  A
// medium triangle becomes one entry per edge of its smaller source-incident pair (times the chunks
// of its other one, when that one is long and the triangle not too large); a heavy one gets
// count chunks of 256 source edges and prefix chunks of 256 edges of one list.  Unit records are
// grouped by their first time and the light and medium lists copied in window-cell order (a
// necessary condition on the pairs' first and last edge times), so that a query with a time
// window visits only what can fall inside it; the results never depend on any of these orders.
// Also the graph totals reported in the statistics: the sum over triangles of the product of the
// three pair multiplicities (the count at infinite deltas, an overflow bound) and the algorithmic
// bytes of one whole-graph count.
#include <algorithm>
#include <cstring>

#include "count_dev.h"

namespace dt {

namespace {

constexpr unsigned kBlock = 256;

__device__ __forceinline__ uint32_t ceil_log2_1(uint32_t s) {   // ceil(log2(s + 1))
    return s == 0 ? 0 : 32 - __clz(s);
}

enum : int { kClsLight = 0, kClsMedium = 1, kClsHeavy = 2, kClsContest = 3 };
constexpr int kClasses = 4;
// the medium path's per-lane counts are 32-bit sums over a wavefront: inner pairs stay below 2^25
constexpr uint64_t kMediumMaxInner = 1ull << 25;
constexpr uint32_t kCrossSample = 128;   // outer edges sampled by the level search

struct SplitRule {
    uint64_t cap_l, cap_m;
    uint32_t force, cost_pct;
};

// The pair budget of a triangle outside the light rule: how many (uv edge, uw edge) pairs the
// medium path may evaluate before its cost passes the prefix procedures' cost times cost_pct / 100.
// Costs are counted in binary-search steps of the searches each path makes: the medium path pays 4
// searches into the inner source pair (or into each chunk of it) per outer edge plus a fixed
// overhead, then about 10 searches into the {v,w} lists per close pair; the prefix procedures pay per source edge 14 searches into
// the other source pair and 24 into the {v,w} lists (prefix and count passes) plus an overhead.
__device__ __forceinline__ double pair_budget(uint64_t s_uv, uint64_t s_uw, uint64_t s_vw, uint32_t cost_pct) {
    const double luv = ceil_log2_1((uint32_t)s_uv) + 1.0, luw = ceil_log2_1((uint32_t)s_uw) + 1.0,
                 lvw = ceil_log2_1((uint32_t)s_vw) + 1.0;
    const double heavy = (double)s_uv * (14.0 * luw + 24.0 * lvw + 12.0) + (double)s_uw * (14.0 * luv + 24.0 * lvw + 12.0);
    const bool outer_uv = cdev::medium_outer_is_uv((uint32_t)s_uv, (uint32_t)s_uw);
    const uint32_t chunks = cdev::medium_inner_chunks((uint32_t)(outer_uv ? s_uv : s_uw), (uint32_t)(outer_uv ? s_uw : s_uv));
    const double lin = chunks > 1 ? ceil_log2_1(cdev::kInnerChunk) + 1.0 : (outer_uv ? luw : luv);
    const double outer = (double)(outer_uv ? s_uv : s_uw) * chunks * (4.0 * lin + 8.0);
    return (heavy * cost_pct / 100.0 - outer) / (10.0 * lvw + 6.0);
}

// class of a triangle that is no unit record: light, always medium, always heavy, or contested
__device__ __forceinline__ int tri_class(uint64_t s_uv, uint64_t s_uw, uint64_t s_vw, const SplitRule &R) {
    const uint64_t P = s_uv * s_uw;
    if (R.force == 1) return kClsLight;
    if (R.force == 2) return kClsHeavy;
    if (R.force == 3) return P < (1ull << 31) && s_uv < kMediumMaxInner && s_uw < kMediumMaxInner ? kClsMedium : kClsHeavy;
    if (P <= R.cap_l && s_vw <= cdev::kLightVw) return kClsLight;
    if (P > R.cap_m || s_uv >= kMediumMaxInner || s_uw >= kMediumMaxInner) return kClsHeavy;
    const double B = pair_budget(s_uv, s_uw, s_vw, R.cost_pct);
    if (B < 0.0) return kClsHeavy;
    if ((double)P <= B) return kClsMedium;
    return kClsContest;
}

constexpr int kSumWords = 5;   // sum_sigma3 lo, hi, bytes, light, medium bytes
constexpr int kTotWords = kClasses + kSumWords;   // class sizes, then the sums

// What the passes of a schedule count into, zeroed together.
struct SchedCtr {
    unsigned long long tot[kTotWords];         // k_classify's totals
    unsigned long long units[16], rest[16];    // k_unit_split's counters (a line each, [0] used)
    unsigned long long ticket[16];             // k_classify blocks done
    unsigned long long cls_n[kClasses][16];    // k_partition's places
    unsigned long long hist[2][kCells];        // light, medium triangles of each window cell
    unsigned long long cur[2][kCells];         // and places taken in it
    unsigned long long lev_hist[kLevels], lev_cur[kLevels];   // contested triangles of each level
};

// Per list entry its class (one byte; kClasses for an empty entry), and the totals: class sizes, the
// sum of sigma products (128-bit) and byte totals.  The list has *n_p entries (at most n_max; null:
// n_max).  A block adds its sums with one atomic each and the block that comes last writes the
// totals and the split's counters to the host, so that no pass over per-block sums and no copy
// follows.
__global__ void __launch_bounds__(kBlock)
k_classify(uint64_t n_max, const unsigned long long *__restrict__ n_p, const uint32_t *__restrict__ tri,
           const uint32_t *__restrict__ eoff, SplitRule R, uint8_t *__restrict__ cls, SchedCtr *__restrict__ ctr,
           unsigned long long *__restrict__ host) {
    __shared__ unsigned long long s_w[kSumWords][kBlock / 64];
    __shared__ unsigned s_cnt[kClasses], s_last;
    if (threadIdx.x < kClasses) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t n_tri = n_p && *n_p < n_max ? *n_p : n_max;
    unsigned __int128 acc = 0;
    unsigned long long bytes = 0, bytes_light = 0, bytes_medium = 0;
    unsigned c[kClasses] = {0, 0, 0, 0};
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n_tri; i += (uint64_t)gridDim.x * kBlock) {
        const uint32_t e_uv = tri[3 * i], e_uw = tri[3 * i + 1], e_vw = tri[3 * i + 2];
        if (e_uv == kNoEdge) {   // an empty entry: no class
            cls[i] = (uint8_t)kClasses;
            continue;
        }
        const uint64_t s_uv = eoff[2 * e_uv + 2] - eoff[2 * e_uv];
        const uint64_t s_uw = eoff[2 * e_uw + 2] - eoff[2 * e_uw];
        const uint32_t s_vw = eoff[2 * e_vw + 2] - eoff[2 * e_vw];
        const int k = tri_class(s_uv, s_uw, s_vw, R);
        cls[i] = (uint8_t)k;
#pragma unroll
        for (int x = 0; x < kClasses; ++x) c[x] += k == x;
        acc += (unsigned __int128)(s_uv * s_uw) * s_vw;
        const uint32_t probe = 2 * ceil_log2_1(s_vw);
        const uint64_t b = 12 + 36 + 8 * (s_uv + s_uw) + 8 * (uint64_t)(s_vw < probe ? s_vw : probe);
        bytes += b;
        bytes_light += k == kClsLight ? b : 0;
        bytes_medium += (k == kClsMedium || k == kClsContest) ? b : 0;
    }
#pragma unroll
    for (int x = 0; x < kClasses; ++x)
        if (c[x]) atomicAdd(&s_cnt[x], c[x]);
    // block sums: within each wavefront by shuffles (the 128-bit sum as two words with carry), then
    // over the wavefronts
    unsigned long long lo = (unsigned long long)acc, hi = (unsigned long long)(acc >> 64);
    unsigned long long w[kSumWords - 2] = {bytes, bytes_light, bytes_medium};
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long lo2 = __shfl_xor(lo, o, 64), hi2 = __shfl_xor(hi, o, 64);
        const unsigned long long s = lo + lo2;
        hi += hi2 + (s < lo ? 1ull : 0ull);
        lo = s;
#pragma unroll
        for (int x = 0; x < kSumWords - 2; ++x) w[x] += __shfl_xor(w[x], o, 64);
    }
    const unsigned wave = threadIdx.x / 64;
    if ((threadIdx.x & 63) == 0) {
        s_w[0][wave] = lo;
        s_w[1][wave] = hi;
        for (int x = 2; x < kSumWords; ++x) s_w[x][wave] = w[x - 2];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned __int128 t = 0;
        unsigned long long tw[kSumWords] = {0, 0, 0, 0, 0};
        for (unsigned j = 0; j < kBlock / 64; ++j) {
            t += ((unsigned __int128)s_w[1][j] << 64) | s_w[0][j];
            for (int x = 2; x < kSumWords; ++x) tw[x] += s_w[x][j];
        }
        for (int x = 0; x < kClasses; ++x)
            if (s_cnt[x]) atomicAdd(&ctr->tot[x], (unsigned long long)s_cnt[x]);
        const unsigned long long t0 = (unsigned long long)t;
        unsigned long long t1 = (unsigned long long)(t >> 64);
        if (t0) t1 += atomicAdd(&ctr->tot[kClasses], t0) + t0 < t0 ? 1ull : 0ull;
        if (t1) atomicAdd(&ctr->tot[kClasses + 1], t1);
        for (int x = 2; x < kSumWords; ++x)
            if (tw[x]) atomicAdd(&ctr->tot[kClasses + x], tw[x]);
        __threadfence();
        s_last = atomicAdd(&ctr->ticket[0], 1ull) == gridDim.x - 1;
    }
    __syncthreads();
    if (s_last) {
        __threadfence();
        if (threadIdx.x < kTotWords)
            host[threadIdx.x] = __hip_atomic_load(&ctr->tot[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else if (threadIdx.x == kTotWords) host[kTotWords] = ctr->units[0];
        else if (threadIdx.x == kTotWords + 1) host[kTotWords + 1] = ctr->rest[0];
    }
}

// Window cell of a light or medium triangle: slice of F (the latest first-edge time over its three
// pairs) times kSlices plus slice of L (the earliest last-edge time).  Each pair's two direction
// lists are key-sorted, so its first and last edges are at their ends.
__device__ __forceinline__ uint16_t window_cell(uint32_t e_uv, uint32_t e_uw, uint32_t e_vw,
                                                const uint32_t *__restrict__ eoff,
                                                const uint64_t *__restrict__ key, int shift, int cshift) {
    const uint32_t es[3] = {e_uv, e_uw, e_vw};
    uint64_t F = 0, L = ~0ull;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const uint32_t a = eoff[2 * es[p]], b = eoff[2 * es[p] + 1], c = eoff[2 * es[p] + 2];
        uint64_t first = ~0ull, last = 0;
        if (a < b) {
            first = key[a];
            last = key[b - 1];
        }
        if (b < c) {
            first = key[b] < first ? key[b] : first;
            last = key[c - 1] > last ? key[c - 1] : last;
        }
        F = first > F ? first : F;
        L = last < L ? last : L;
    }
    const uint64_t f = (F >> shift) >> cshift, l = (L >> shift) >> cshift;
    return (uint16_t)((f < kSlices - 1 ? f : kSlices - 1) * kSlices + (l < kSlices - 1 ? l : kSlices - 1));
}

// Per DAG edge with one temporal edge: that edge's key, with its direction (1: head -> tail) in
// bit 63, which is free while unit records are built (spans below 2^31 and fewer than 2^31 edges
// keep keys below 2^62); all ones for other edges.
__global__ void k_unit_keys(uint64_t ms, const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key,
                            uint64_t *__restrict__ ukey) {
    const uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= ms) return;
    const uint32_t a = eoff[2 * e], b = eoff[2 * e + 1], c = eoff[2 * e + 2];
    ukey[e] = c - a == 1 ? key[a] | (uint64_t)(a == b ? 1u : 0u) << 63 : ~0ull;
}

// Unit triangles out of the list: the three unit keys of an entry say whether it is one and make its
// record (with its t1 bucket as a sort key); the other triangles go to the rest list.  A workgroup
// holds a tile of kSplitPer entries a thread, all their gathers in flight together, and takes the
// tile's places in both outputs with one atomic each.  Bound by the list and the gathers of the third
// edges' keys; one pass where classifying every entry and then moving it read both twice (67M entries:
// classify 1.0 and partition 1.9 ms, this pass 1.0; the whole schedule 4.7 -> 2.9 ms).  Past unit_cap and
// rest_cap triangles are counted and not written.
constexpr unsigned kSplitPer = 8;
constexpr unsigned kSplitTile = kBlock * kSplitPer;
__global__ void __launch_bounds__(kBlock)
k_unit_split(uint64_t nt, const uint32_t *__restrict__ tri, const uint64_t *__restrict__ ukey, int shift, int bshift,
             uint4 *__restrict__ urec, uint16_t *__restrict__ ubkt, uint64_t unit_cap,
             uint32_t *__restrict__ rest, uint64_t rest_cap,
             SchedCtr *__restrict__ ctr) {
    __shared__ uint32_t s_cnt[2][kBlock / 64];
    __shared__ unsigned long long s_base[2];
    const unsigned lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const uint64_t below = (1ull << lane) - 1;
    for (uint64_t t0 = (uint64_t)blockIdx.x * kSplitTile; t0 < nt; t0 += (uint64_t)gridDim.x * kSplitTile) {
        uint32_t e[kSplitPer][3];
        uint64_t k[kSplitPer][3];
#pragma unroll
        for (unsigned j = 0; j < kSplitPer; ++j) {
            const uint64_t i = t0 + j * kBlock + threadIdx.x;
#pragma unroll
            for (int x = 0; x < 3; ++x) e[j][x] = i < nt ? tri[3 * i + x] : kNoEdge;
        }
#pragma unroll
        for (unsigned j = 0; j < kSplitPer; ++j)
#pragma unroll
            for (int x = 0; x < 3; ++x) k[j][x] = e[j][0] != kNoEdge ? ukey[e[j][x]] : ~0ull;
        uint32_t nu = 0, nr = 0;   // of this wavefront
#pragma unroll
        for (unsigned j = 0; j < kSplitPer; ++j) {
            const bool unit = k[j][0] != ~0ull && k[j][1] != ~0ull && k[j][2] != ~0ull;
            nu += (uint32_t)__popcll(__ballot(unit));
            nr += (uint32_t)__popcll(__ballot(!unit && e[j][0] != kNoEdge));
        }
        if (lane == 0) {
            s_cnt[0][wave] = nu;
            s_cnt[1][wave] = nr;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            uint32_t n = 0;
            for (unsigned w = 0; w < kBlock / 64; ++w) {
                const uint32_t c = s_cnt[threadIdx.x][w];
                s_cnt[threadIdx.x][w] = n;
                n += c;
            }
            s_base[threadIdx.x] = n ? atomicAdd(threadIdx.x ? ctr->rest : ctr->units, (unsigned long long)n) : 0ull;
        }
        __syncthreads();
        uint64_t pu = s_base[0] + s_cnt[0][wave], pr = s_base[1] + s_cnt[1][wave];
#pragma unroll
        for (unsigned j = 0; j < kSplitPer; ++j) {
            const bool unit = k[j][0] != ~0ull && k[j][1] != ~0ull && k[j][2] != ~0ull;
            const bool other = !unit && e[j][0] != kNoEdge;
            const uint64_t um = __ballot(unit), rm = __ballot(other);
            if (unit) {
                const uint64_t p = pu + (uint32_t)__popcll(um & below);
                const uint64_t k3[3] = {k[j][0] & ~(1ull << 63), k[j][1] & ~(1ull << 63), k[j][2] & ~(1ull << 63)};
                const int d3[3] = {(int)(k[j][0] >> 63), (int)(k[j][1] >> 63), (int)(k[j][2] >> 63)};
                const uint4 r = cdev::unit_record_of(k3, d3, shift);
                if (p < unit_cap) {
                    urec[p] = r;
                    ubkt[p] = (uint16_t)(r.x >> bshift);
                }
            }
            if (other) {
                const uint64_t p = pr + (uint32_t)__popcll(rm & below);
                if (p < rest_cap) {
                    rest[3 * p] = e[j][0];
                    rest[3 * p + 1] = e[j][1];
                    rest[3 * p + 2] = e[j][2];
                }
            }
            pu += (uint32_t)__popcll(um);
            pr += (uint32_t)__popcll(rm);
        }
    }
}

// Every triangle to its class's list: light and always-medium triangles with their window cells (mcell:
// the always-medium ones first, then the n_c contested ones), which are counted too; always-heavy ones
// after the n_c contested ones in the heavy list; contested ones to crec for the level search.  A
// workgroup takes its tile's places in each list with one atomic a class.
constexpr unsigned kPartPer = 4;
constexpr unsigned kPartTile = kBlock * kPartPer;
__global__ void __launch_bounds__(kBlock)
k_partition(uint64_t n_tri, const uint32_t *__restrict__ tri, const uint8_t *__restrict__ cls,
            const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key, int shift, int cshift, uint64_t n_a,
            uint64_t n_c, uint32_t *__restrict__ light, uint32_t *__restrict__ medium, uint32_t *__restrict__ heavy,
            uint4 *__restrict__ crec, uint16_t *__restrict__ lcell, uint16_t *__restrict__ mcell,
            SchedCtr *__restrict__ ctr) {
    __shared__ uint32_t s_hist[2][kCells];
    __shared__ uint32_t s_cnt[kClasses][kBlock / 64];
    __shared__ unsigned long long s_base[kClasses];
    const unsigned lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const uint64_t below = (1ull << lane) - 1;
    for (unsigned x = threadIdx.x; x < 2 * kCells; x += kBlock) s_hist[x / kCells][x % kCells] = 0;
    for (uint64_t t0 = (uint64_t)blockIdx.x * kPartTile; t0 < n_tri; t0 += (uint64_t)gridDim.x * kPartTile) {
        int k[kPartPer];
        uint32_t mine[kClasses] = {0, 0, 0, 0};   // of this wavefront
#pragma unroll
        for (unsigned j = 0; j < kPartPer; ++j) {
            const uint64_t i = t0 + j * kBlock + threadIdx.x;
            k[j] = i < n_tri ? cls[i] : kClasses;
        }
#pragma unroll
        for (unsigned j = 0; j < kPartPer; ++j)
#pragma unroll
            for (int c = 0; c < kClasses; ++c) mine[c] += (uint32_t)__popcll(__ballot(k[j] == c));
        __syncthreads();   // (s_hist zeroed; the last tile's places read)
        if (lane == 0)
            for (int c = 0; c < kClasses; ++c) s_cnt[c][wave] = mine[c];
        __syncthreads();
        if (threadIdx.x < kClasses) {
            uint32_t n = 0;
            for (unsigned w = 0; w < kBlock / 64; ++w) {
                const uint32_t x = s_cnt[threadIdx.x][w];
                s_cnt[threadIdx.x][w] = n;
                n += x;
            }
            s_base[threadIdx.x] = n ? atomicAdd(&ctr->cls_n[threadIdx.x][0], (unsigned long long)n) : 0ull;
        }
        __syncthreads();
        uint64_t at[kClasses];
#pragma unroll
        for (int c = 0; c < kClasses; ++c) at[c] = s_base[c] + s_cnt[c][wave];
#pragma unroll
        for (unsigned j = 0; j < kPartPer; ++j) {
            uint64_t pos = 0;
#pragma unroll
            for (int c = 0; c < kClasses; ++c) {
                const uint64_t m = __ballot(k[j] == c);
                if (k[j] == c) pos = at[c] + (uint32_t)__popcll(m & below);
                at[c] += (uint32_t)__popcll(m);
            }
            if (k[j] < kClasses) {
                const uint64_t i = t0 + j * kBlock + threadIdx.x;
                const uint32_t e_uv = tri[3 * i], e_uw = tri[3 * i + 1], e_vw = tri[3 * i + 2];
                if (k[j] == kClsContest) {
                    crec[pos] = make_uint4(e_uv, e_uw, e_vw, 0u);
                } else {
                    uint32_t *dst = (k[j] == kClsLight ? light : (k[j] == kClsMedium ? medium : heavy + 3 * n_c)) + 3 * pos;
                    dst[0] = e_uv;
                    dst[1] = e_uw;
                    dst[2] = e_vw;
                }
                if (k[j] != kClsHeavy) {
                    const uint16_t cell = window_cell(e_uv, e_uw, e_vw, eoff, key, shift, cshift);
                    if (k[j] == kClsLight) lcell[pos] = cell;
                    else mcell[k[j] == kClsContest ? n_a + pos : pos] = cell;
                    atomicAdd(&s_hist[k[j] == kClsLight ? 0 : 1][cell], 1u);
                }
            }
        }
    }
    __syncthreads();
    for (unsigned x = threadIdx.x; x < 2 * kCells; x += kBlock) {
        const uint32_t n = s_hist[x / kCells][x % kCells];
        if (n) atomicAdd(&ctr->hist[x / kCells][x % kCells], (unsigned long long)n);
    }
}

// Level of every contested triangle (one wavefront each): the largest l in 1..kLevels-1 whose
// close pairs -- (x, y) with x on the outer source pair, y on the inner one, |t_x - t_y| <= D(l),
// both directions of both pairs, the whole span -- are at most the triangle's pair budget, or 0.
// The close pairs are counted exactly (two binary searches per outer edge and inner direction) on
// up to kCrossSample outer edges spread evenly over the pair and scaled to all of them, stopping
// once the budget is passed; the levels are found by binary search (close pairs grow with D).
// Writes the level to crec[i].w and counts the triangles of each level.  The level only
// decides which exact method counts the triangle for a query.
__global__ void __launch_bounds__(kBlock)
k_crossover(uint64_t nc, uint4 *__restrict__ crec, const uint32_t *__restrict__ eoff,
            const uint64_t *__restrict__ key, int shift, int64_t span, uint32_t cost_pct, SchedCtr *__restrict__ ctr) {
    __shared__ uint32_t s_lev[kLevels];
    if (threadIdx.x < kLevels) s_lev[threadIdx.x] = 0;
    __syncthreads();
    const unsigned lane = threadIdx.x & 63;
    const uint64_t nw = (uint64_t)gridDim.x * (kBlock / 64);
    for (uint64_t i = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / 64; i < nc; i += nw) {
        const uint4 r = crec[i];
        const uint32_t a0 = eoff[2 * r.x], a1 = eoff[2 * r.x + 1], a2 = eoff[2 * r.x + 2];
        const uint32_t b0 = eoff[2 * r.y], b1 = eoff[2 * r.y + 1], b2 = eoff[2 * r.y + 2];
        const uint64_t s_vw = eoff[2 * r.z + 2] - eoff[2 * r.z];
        const double B = pair_budget(a2 - a0, b2 - b0, s_vw, cost_pct);
        const bool outer_uv = cdev::medium_outer_is_uv(a2 - a0, b2 - b0);
        const uint32_t o0 = outer_uv ? a0 : b0, o2 = outer_uv ? a2 : b2;
        const uint32_t i0 = outer_uv ? b0 : a0, i1 = outer_uv ? b1 : a1, i2 = outer_uv ? b2 : a2;
        auto bound = [&](int64_t x) -> uint64_t {   // key bound of "t < x" (relative times)
            return x <= 0 ? 0ull : (x > span ? ~0ull : ((uint64_t)x << shift));
        };
        const uint32_t n_out = o2 - o0;
        const uint32_t n_s = n_out < kCrossSample ? n_out : kCrossSample;
        const double scale = n_s ? (double)n_out / n_s : 0.0;
        // within the budget at distance D (the same answer in every lane)
        auto fits = [&](int64_t D) -> bool {
            unsigned long long c = 0;
            for (uint32_t s0 = 0; s0 < n_s; s0 += 64) {
                const uint32_t si = s0 + lane;
                if (si < n_s) {
                    const uint32_t x = o0 + (uint32_t)(((uint64_t)si * n_out) / n_s);
                    const int64_t tx = (int64_t)(key[x] >> shift);
                    const uint64_t klo = bound(tx - D), khi = bound(tx + D + 1);
                    uint32_t l0, h0, l1, h1;
                    cdev::lower2(key, i0, i1, klo, khi, l0, h0);
                    cdev::lower2(key, i1, i2, klo, khi, l1, h1);
                    c += (h0 - l0) + (h1 - l1);
                }
                if ((double)cdev::wave_sum(c) * scale > B) return false;
            }
            return true;
        };
        uint32_t lo = 0, hi = kLevels - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) / 2;
            if (fits(level_delta(mid))) lo = mid;
            else hi = mid - 1;
        }
        if (lane == 0) {
            crec[i].w = lo;
            atomicAdd(&s_lev[lo], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < kLevels && s_lev[threadIdx.x])
        atomicAdd(&ctr->lev_hist[threadIdx.x], (unsigned long long)s_lev[threadIdx.x]);
}

// Exclusive sums over the workgroup of one value a thread, in thread order; the total to every thread.
__device__ __forceinline__ unsigned long long block_scan(unsigned long long v, unsigned long long *s_wave,
                                                         unsigned long long &total) {
    const unsigned lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    unsigned long long x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(x, o, 64);
        if (lane >= (unsigned)o) x += y;
    }
    __syncthreads();   // (the last call's s_wave read)
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    unsigned long long before = 0;
    total = 0;
    for (unsigned w = 0; w < blockDim.x / 64; ++w) {
        before += w < wave ? s_wave[w] : 0ull;
        total += s_wave[w];
    }
    return before + x - v;
}

// Starts of the window cells in a list, from its triangles of each cell.
__device__ __forceinline__ void cell_starts(const unsigned long long *__restrict__ hist, unsigned long long *s_start,
                                            unsigned long long *s_wave) {
    constexpr unsigned per = kCells / kBlock;
    static_assert(kCells % kBlock == 0, "cells a thread");
    unsigned long long h[per], n = 0, total;
#pragma unroll
    for (unsigned x = 0; x < per; ++x) {
        h[x] = hist[per * threadIdx.x + x];
        n += h[x];
    }
    unsigned long long at = block_scan(n, s_wave, total);
#pragma unroll
    for (unsigned x = 0; x < per; ++x) {
        s_start[per * threadIdx.x + x] = at;
        at += h[x];
    }
}

// The windowed copies in window-cell order, and the contested triangles in descending level order:
// after the n_a always-medium ones in the medium list and first in the heavy list.  Tiles of the light
// list, of the always-medium list and of crec, one a workgroup: ranks within a tile by atomics in LDS,
// the tile's places in a cell (and level) with one atomic each.  The order within a cell is of no
// matter, so this takes the place of three sorts with their temporaries and the passes that packed and
// unpacked their records (86 us for the lists of 61M edges).
constexpr unsigned kPlacePer = 8;
constexpr unsigned kPlaceTile = kBlock * kPlacePer;
__global__ void __launch_bounds__(kBlock)
k_place(uint64_t n_l, uint64_t n_a, uint64_t n_c, unsigned tiles_l, unsigned tiles_a, const uint32_t *__restrict__ light,
        const uint16_t *__restrict__ lcell, uint32_t *__restrict__ medium, const uint16_t *__restrict__ mcell,
        const uint4 *__restrict__ crec, uint32_t *__restrict__ heavy, uint32_t *__restrict__ light_w,
        uint32_t *__restrict__ medium_w, uint8_t *__restrict__ mlev_w, SchedCtr *__restrict__ ctr) {
    __shared__ unsigned long long s_at[kCells], s_lat[kLevels], s_wave[kBlock / 64];
    __shared__ uint32_t s_cnt[kCells], s_lcnt[kLevels];
    const int seg = blockIdx.x < tiles_l ? 0 : (blockIdx.x < tiles_l + tiles_a ? 1 : 2);
    const uint64_t n = seg == 0 ? n_l : (seg == 1 ? n_a : n_c);
    const uint64_t t0 = (uint64_t)(blockIdx.x - (seg == 0 ? 0u : (seg == 1 ? tiles_l : tiles_l + tiles_a))) * kPlaceTile;
    const uint16_t *cells = seg == 0 ? lcell : (seg == 1 ? mcell : mcell + n_a);
    const int list = seg == 0 ? 0 : 1;
    for (unsigned x = threadIdx.x; x < kCells; x += kBlock) s_cnt[x] = 0;
    if (threadIdx.x < kLevels) s_lcnt[threadIdx.x] = 0;
    cell_starts(ctr->hist[list], s_at, s_wave);
    __syncthreads();
    uint32_t cell[kPlacePer], rank[kPlacePer], lrank[kPlacePer];
    uint4 r[kPlacePer];
#pragma unroll
    for (unsigned j = 0; j < kPlacePer; ++j) {
        const uint64_t i = t0 + j * kBlock + threadIdx.x;
        cell[j] = kCells;
        if (i < n) {
            cell[j] = cells[i];
            if (seg == 2) {
                r[j] = crec[i];
            } else {
                const uint32_t *src = (seg == 0 ? light : medium) + 3 * i;
                r[j] = make_uint4(src[0], src[1], src[2], (uint32_t)kLevelAlways);
            }
        }
    }
#pragma unroll
    for (unsigned j = 0; j < kPlacePer; ++j)
        if (cell[j] < kCells) {
            rank[j] = atomicAdd(&s_cnt[cell[j]], 1u);
            if (seg == 2) lrank[j] = atomicAdd(&s_lcnt[r[j].w], 1u);
        }
    __syncthreads();
    for (unsigned x = threadIdx.x; x < kCells; x += kBlock)
        if (s_cnt[x]) s_at[x] += atomicAdd(&ctr->cur[list][x], (unsigned long long)s_cnt[x]);
    if (seg == 2 && threadIdx.x < kLevels && s_lcnt[threadIdx.x]) {
        unsigned long long above = 0;   // contested triangles of higher levels
        for (unsigned l = threadIdx.x + 1; l < kLevels; ++l) above += ctr->lev_hist[l];
        s_lat[threadIdx.x] = above + atomicAdd(&ctr->lev_cur[threadIdx.x], (unsigned long long)s_lcnt[threadIdx.x]);
    }
    __syncthreads();
#pragma unroll
    for (unsigned j = 0; j < kPlacePer; ++j)
        if (cell[j] < kCells) {
            const uint64_t p = s_at[cell[j]] + rank[j];
            uint32_t *dst = (seg == 0 ? light_w : medium_w) + 3 * p;
            dst[0] = r[j].x;
            dst[1] = r[j].y;
            dst[2] = r[j].z;
            if (seg != 0) mlev_w[p] = (uint8_t)r[j].w;
            if (seg == 2) {
                const uint64_t c = s_lat[r[j].w] + lrank[j];
                uint32_t *m = medium + 3 * (n_a + c), *h = heavy + 3 * c;
                m[0] = h[0] = r[j].x;
                m[1] = h[1] = r[j].y;
                m[2] = h[2] = r[j].z;
            }
        }
}

// first position of every bucket 0..nbk in the nu sorted bucket keys (a binary search per bucket;
// nu for nbk and for buckets past the last key)
__global__ void k_unit_starts(uint64_t nu, uint32_t nbk, const uint16_t *__restrict__ bkt,
                              uint32_t *__restrict__ start) {
    const uint32_t x = blockIdx.x * kBlock + threadIdx.x;
    if (x > nbk) return;
    uint64_t lo = 0, len = nu;
    while (len > 0) {
        const uint64_t half = len >> 1;
        if (bkt[lo + half] < x) {
            lo += half + 1;
            len -= half + 1;
        } else {
            len = half;
        }
    }
    start[x] = (uint32_t)lo;
}

constexpr uint32_t kChunk = 256;   // source edges per count chunk and per prefix chunk

// Work items of the medium and heavy lists, in three launches for all of them: sizes and their sums a
// tile (k_sizes), the sums' prefix over the tiles (k_tile_sums), and in k_expand the prefix within the
// tile and the items, which a tile writes in order, each thread finding its item's triangle in the
// tile's prefix (one triangle a thread wrote them scattered: 60 us for both medium lists of the 10M-edge
// graph, 27 us so with the heavy ones).  A tile of many items is shared by several workgroups, as few
// tiles otherwise leave most of the chip idle (34,220 triangles of 300 items each: schedule 490 us, 1,450
// with a workgroup a tile).  Five sequences: the medium entries of medium and of medium_w (one
// per edge of the outer pair, the source-incident pair with fewer temporal edges, and chunk of the inner
// pair), then of the heavy triangles the prefix slots (four arrays of length sigma + 1), count chunks and
// prefix chunks (at least one per list, so that an empty list's total is written too).
constexpr unsigned kItemPer = 4;
constexpr unsigned kItemTile = kBlock * kItemPer;
constexpr int kSeqs = 5;
constexpr uint64_t kItemsPerBlock = 8192;
struct ItemArgs {
    uint64_t nm, nh;
    unsigned tiles_m, tiles_h;   // (each list + 1 entry, so that the last prefix is the total)
    const uint32_t *eoff, *medium, *medium_w, *heavy;
    unsigned long long *size[4];    // of medium, medium_w, slots, prefix chunks
    unsigned long long *base[kSeqs];   // first item (n + 1 entries)
    unsigned long long *tile;       // [kSeqs][max tiles]
    unsigned tile_stride;
    uint32_t *mitems, *mitems_w, *chunks, *pchunks;
};

__device__ __forceinline__ uint64_t medium_size(const uint32_t *__restrict__ med, uint64_t i,
                                                const uint32_t *__restrict__ eoff) {
    const uint32_t e_uv = med[3 * i], e_uw = med[3 * i + 1];
    const uint32_t s_uv = eoff[2 * e_uv + 2] - eoff[2 * e_uv], s_uw = eoff[2 * e_uw + 2] - eoff[2 * e_uw];
    const bool outer_uv = cdev::medium_outer_is_uv(s_uv, s_uw);
    const uint32_t s_out = outer_uv ? s_uv : s_uw, s_in = outer_uv ? s_uw : s_uv;
    return (uint64_t)s_out * cdev::medium_inner_chunks(s_out, s_in);
}

// lengths of a heavy triangle's four source lists: uv out, uv in, uw out, uw in
__device__ __forceinline__ void heavy_lens(const uint32_t *__restrict__ heavy, uint64_t h,
                                           const uint32_t *__restrict__ eoff, uint32_t len[4]) {
    const uint32_t e_uv = heavy[3 * h], e_uw = heavy[3 * h + 1];
    len[0] = eoff[2 * e_uv + 1] - eoff[2 * e_uv];
    len[1] = eoff[2 * e_uv + 2] - eoff[2 * e_uv + 1];
    len[2] = eoff[2 * e_uw + 1] - eoff[2 * e_uw];
    len[3] = eoff[2 * e_uw + 2] - eoff[2 * e_uw + 1];
}

__device__ __forceinline__ uint64_t list_chunks(uint32_t len) { return len ? ((uint64_t)len + kChunk - 1) / kChunk : 1; }

__global__ void __launch_bounds__(kBlock) k_sizes(ItemArgs A) {
    __shared__ unsigned long long s_sum[3];
    if (threadIdx.x < 3) s_sum[threadIdx.x] = 0;
    __syncthreads();
    const bool med = blockIdx.x < A.tiles_m;
    const unsigned tile = med ? blockIdx.x : blockIdx.x - A.tiles_m;
    unsigned long long sum[3] = {0, 0, 0};
    for (unsigned j = 0; j < kItemPer; ++j) {
        const uint64_t i = (uint64_t)tile * kItemTile + j * kBlock + threadIdx.x;
        if (med && i <= A.nm) {
            const uint64_t x = i < A.nm ? medium_size(A.medium, i, A.eoff) : 0;
            const uint64_t y = i < A.nm ? medium_size(A.medium_w, i, A.eoff) : 0;
            A.size[0][i] = x;
            A.size[1][i] = y;
            sum[0] += x;
            sum[1] += y;
        } else if (!med && i <= A.nh) {
            uint64_t slots = 0, p = 0;
            if (i < A.nh) {
                uint32_t len[4];
                heavy_lens(A.heavy, i, A.eoff, len);
                slots = (uint64_t)len[0] + len[1] + len[2] + len[3] + 4;
                for (int X = 0; X < 4; ++X) p += list_chunks(len[X]);
            }
            A.size[2][i] = slots;
            A.size[3][i] = p;
            sum[0] += slots;
            sum[1] += slots ? (slots - 4 + kChunk - 1) / kChunk : 0;
            sum[2] += p;
        }
    }
    for (int x = 0; x < 3; ++x) {
        const unsigned long long t = cdev::wave_sum(sum[x]);
        if ((threadIdx.x & 63) == 0 && t) atomicAdd(&s_sum[x], t);
    }
    __syncthreads();
    if (threadIdx.x < (med ? 2u : 3u)) A.tile[(med ? 0 : 2) * A.tile_stride + threadIdx.x * A.tile_stride + tile] = s_sum[threadIdx.x];
}

// One workgroup: the tiles' sums to exclusive prefixes, the totals and the most items of a tile to the host.
constexpr unsigned kTileBlock = 1024;
__global__ void __launch_bounds__(kTileBlock) k_tile_sums(ItemArgs A, unsigned long long *__restrict__ host) {
    __shared__ unsigned long long s_wave[kTileBlock / 64];
    __shared__ unsigned long long s_most;
    if (threadIdx.x == 0) s_most = 0;
    unsigned long long most = 0;
    for (int x = 0; x < kSeqs; ++x) {
        unsigned long long *t = A.tile + (uint64_t)x * A.tile_stride;
        const unsigned n = x < 2 ? A.tiles_m : A.tiles_h;
        unsigned long long run = 0;
        for (unsigned b = 0; b < n; b += kTileBlock) {
            const unsigned i = b + threadIdx.x;
            const unsigned long long v = i < n ? t[i] : 0ull;
            if (x != 2 && v > most) most = v;   // (the slots have no items)
            unsigned long long total;
            const unsigned long long at = block_scan(v, s_wave, total);
            if (i < n) t[i] = run + at;
            run += total;
        }
        if (threadIdx.x == 0) host[x] = run;
    }
    if (most) atomicMax(&s_most, most);
    __syncthreads();
    if (threadIdx.x == 0) host[kSeqs] = s_most;
}

// the tile's item p of s_pre (kItemTile + 1 prefixes): its entry
__device__ __forceinline__ unsigned item_entry(const unsigned long long *s_pre, unsigned long long p) {
    unsigned lo = 0, len = kItemTile;   // the last entry with prefix <= p
    while (len > 1) {
        const unsigned half = len / 2;
        if (s_pre[lo + half] <= p) lo += half;
        len -= half;
    }
    return lo;
}

__global__ void __launch_bounds__(kBlock) k_expand(ItemArgs A) {
    __shared__ unsigned long long s_pre[kItemTile + 1], s_wave[kBlock / 64];
    const bool med = blockIdx.x < A.tiles_m;
    const unsigned tile = med ? blockIdx.x : blockIdx.x - A.tiles_m;
    const uint64_t t0 = (uint64_t)tile * kItemTile, n = med ? A.nm : A.nh;
    for (int x = med ? 0 : 2; x < (med ? 2 : kSeqs); ++x) {
        const unsigned long long *size = A.size[x < 3 ? x : x - 1];
        unsigned long long v[kItemPer], mine = 0, total;
#pragma unroll
        for (unsigned j = 0; j < kItemPer; ++j) {
            const uint64_t i = t0 + kItemPer * threadIdx.x + j;
            v[j] = i <= n ? size[i] : 0ull;
            if (x == 3) v[j] = v[j] ? (v[j] - 4 + kChunk - 1) / kChunk : 0ull;   // count chunks, from the slots
            mine += v[j];
        }
        unsigned long long at = block_scan(mine, s_wave, total);
        const unsigned long long base = A.tile[(uint64_t)x * A.tile_stride + tile];
#pragma unroll
        for (unsigned j = 0; j < kItemPer; ++j) {
            const uint64_t i = t0 + kItemPer * threadIdx.x + j;
            s_pre[kItemPer * threadIdx.x + j] = at;
            if (i <= n && blockIdx.y == 0) A.base[x][i] = base + at;
            at += v[j];
        }
        if (x == 2) continue;   // (the slots have no items)
        if (threadIdx.x == 0) s_pre[kItemTile] = total;
        __syncthreads();
        uint2 *out = reinterpret_cast<uint2 *>(x == 0 ? A.mitems : (x == 1 ? A.mitems_w : (x == 3 ? A.chunks : A.pchunks)));
        const uint64_t step = (uint64_t)gridDim.y * kBlock;
        for (unsigned long long p = (uint64_t)blockIdx.y * kBlock + threadIdx.x; p < total; p += step) {
            const unsigned e = item_entry(s_pre, p);
            uint32_t j = (uint32_t)(p - s_pre[e]);
            if (x == 3) {
                j *= kChunk;
            } else if (x == 4) {
                uint32_t len[4];
                heavy_lens(A.heavy, t0 + e, A.eoff, len);
                uint32_t X = 0;
                while (X < 3 && j >= list_chunks(len[X])) j -= (uint32_t)list_chunks(len[X++]);
                j = j * kChunk | X;
            }
            out[base + p] = make_uint2((uint32_t)(t0 + e), j);
        }
        __syncthreads();   // (s_pre read)
    }
}

// One workgroup, to the host: the cell starts of the light list, the first medium item of every cell, and
// per query level l = 1..kLevels, with c contested triangles of level >= l: the medium entries end at
// those of n_a + c; the heavy triangles, count chunks, prefix chunks and slots start at c.
__global__ void __launch_bounds__(kBlock)
k_tables(uint64_t n_l, uint64_t n_a, ItemArgs A, const SchedCtr *__restrict__ ctr, unsigned long long *__restrict__ host) {
    __shared__ unsigned long long s_at[kCells], s_wave[kBlock / 64];
    cell_starts(ctr->hist[0], s_at, s_wave);
    __syncthreads();
    for (unsigned c = threadIdx.x; c <= kCells; c += kBlock) host[c] = c < kCells ? s_at[c] : n_l;
    __syncthreads();
    cell_starts(ctr->hist[1], s_at, s_wave);
    __syncthreads();
    for (unsigned c = threadIdx.x; c <= kCells; c += kBlock) host[kCells + 1 + c] = A.base[1][c < kCells ? s_at[c] : A.nm];
    const uint32_t l = threadIdx.x;
    if (l == 0 || l > kLevels) return;
    uint64_t c = 0;
    for (uint32_t v = l; v < kLevels; ++v) c += ctr->lev_hist[v];
    unsigned long long *out = host + 2 * (kCells + 1);
    out[0 * (kLevels + 1) + l] = A.base[0][n_a + c];
    out[1 * (kLevels + 1) + l] = c;
    out[2 * (kLevels + 1) + l] = A.base[3][c];
    out[3 * (kLevels + 1) + l] = A.base[4][c];
    out[4 * (kLevels + 1) + l] = A.base[2][c];
}

// One attempt at the schedule.  The unit keys are g's, made here if the build left none.  lean: the
// split's outputs are counted before they are allocated, and with last (nothing reads tri
// afterwards) tri is given back once it is split, so that the attempt holds no more than the
// schedule itself needs.
int try_schedule(dt_graph *g, DevMem &tri, bool with_units, bool last, bool lean) {
    dt_ctx *ctx = g->ctx;
    hipStream_t st = ctx->stream;
    const uint64_t nt = g->n_tri_list;   // list entries (empty ones have no class)
    Schedule &S = g->sched;
    S = Schedule();
    SplitRule R;
    R.cap_l = g->light_cap_used ? g->light_cap_used : 4;
    R.cap_m = g->tuning.medium_pair_cap;
    R.force = g->tuning.force_path;
    R.cost_pct = g->cost_pct_used ? g->cost_pct_used : 100;
    // unit records hold 32-bit relative times
    const bool unit_ok = g->span <= kUnitMaxSpan;
    const bool units = with_units && R.force == 0 && unit_ok && g->m_s && g->n_tri;
    DevMem cls, zero, rest, urec, ubkt;
    DT_TRY(dev_alloc(ctx, zero, sizeof(SchedCtr)));
    SchedCtr *ctr = zero.as<SchedCtr>();
    // t1 buckets of the unit records: at most 2^16, t1 >> unit_shift
    int t_bits = 0;
    while (t_bits < 31 && (1ll << t_bits) <= g->span) ++t_bits;
    S.unit_shift = t_bits > 16 ? t_bits - 16 : 0;
    const uint64_t nbk = unit_ok ? ((uint64_t)g->span >> S.unit_shift) + 1 : 1;
    if (units && !g->ukey.ptr) {
        DT_TRY(dev_alloc(ctx, g->ukey, g->m_s * 8));
        unit_keys(g, st);
        DT_HIP(hipGetLastError());
    }
    // room for unit records of every triangle; for other triangles as many in lists up to 4M (48 MB;
    // a second pass cost 60 us of the 10M-edge graph's build, whose triangles are nearly all others),
    // a quarter of them in longer ones (a twelfth is needed at 61M edges).  The pass runs again at the
    // counted sizes where that is too little.
    uint64_t unit_cap = lean ? 0 : g->n_tri;
    uint64_t rest_cap = lean ? 0 : std::max<uint64_t>(g->n_tri / 4, std::min<uint64_t>(g->n_tri, 1ull << 22));
    uint64_t n_rest = nt;
    unsigned long long *hs = reinterpret_cast<unsigned long long *>(ctx->pinned_stage);
    for (int attempt = 0;; ++attempt) {
        const uint32_t *list = tri.as<uint32_t>();
        if (units) {
            DT_TRY(dev_alloc(ctx, urec, unit_cap * sizeof(uint4)));
            DT_TRY(dev_alloc(ctx, ubkt, unit_cap * 2));
            DT_TRY(dev_alloc(ctx, rest, rest_cap * 12));
            list = rest.as<uint32_t>();
        }
        DT_HIP(hipMemsetAsync(ctr, 0, sizeof(SchedCtr), st));
        if (units) {
            const unsigned sgrid = std::min<unsigned>(grid_for(nt, kSplitTile), (unsigned)ctx->num_cus * 16);
            k_unit_split<<<sgrid, kBlock, 0, st>>>(nt, tri.as<uint32_t>(), g->ukey.as<uint64_t>(), g->shift, S.unit_shift,
                                                   urec.as<uint4>(), ubkt.as<uint16_t>(), unit_cap, rest.as<uint32_t>(),
                                                   rest_cap, ctr);
            DT_HIP(hipGetLastError());
        }
        const uint64_t n_max = units ? rest_cap : nt;
        DT_TRY(dev_alloc(ctx, cls, n_max + 1));
        const unsigned grid = std::min(grid_for(n_max + 1, kBlock * 4), (unsigned)ctx->num_cus * 4);
        k_classify<<<grid, kBlock, 0, st>>>(n_max, units ? ctr->rest : nullptr, list, g->eoff.as<uint32_t>(), R,
                                            cls.as<uint8_t>(), ctr, hs);
        DT_HIP(hipGetLastError());
        DT_HIP(hipStreamSynchronize(st));
        if (!units) break;
        n_rest = hs[kTotWords + 1];
        if (hs[kTotWords] + n_rest != g->n_tri) return fail(DT_EDEVICE, "unit and other triangles do not add up");
        if (hs[kTotWords] <= unit_cap && n_rest <= rest_cap) break;
        if (attempt) return fail(DT_EDEVICE, "triangle classes changed between passes");
        unit_cap = hs[kTotWords];
        rest_cap = n_rest;
    }
    if (units && lean && last) {
        g->ukey.reset();
        tri.reset();
    }
    const uint32_t *list = units ? rest.as<uint32_t>() : tri.as<uint32_t>();
    const uint64_t nu = units ? hs[kTotWords] : 0;
    uint64_t ncls[kClasses];
    for (int c = 0; c < kClasses; ++c) ncls[c] = hs[c];
    const unsigned __int128 s3 = ((unsigned __int128)hs[kClasses + 1] << 64) | hs[kClasses];
    g->sum_sigma3 = s3 + nu;
    g->alg_bytes_unit = sizeof(uint4) * nu;
    g->alg_bytes = hs[kClasses + 2] + g->alg_bytes_unit;
    g->alg_bytes_light = hs[kClasses + 3];
    g->alg_bytes_medium = hs[kClasses + 4];
    const uint64_t na = ncls[kClsMedium], nh_always = ncls[kClsHeavy], nc = ncls[kClsContest];
    if (ncls[kClsLight] + na + nh_always + nu + nc != g->n_tri)
        return fail(DT_EDEVICE, "triangle classes do not add up");
    S.n_light = ncls[kClsLight];
    S.n_always_medium = na;
    S.n_contested = nc;
    S.n_always_heavy = nh_always;
    S.n_medium = na + nc;
    S.n_heavy = nc + nh_always;
    S.n_unit = nu;
    const uint64_t nm = S.n_medium, nh = S.n_heavy;
    DT_TRY(dev_alloc(ctx, S.light, S.n_light * 12));
    DT_TRY(dev_alloc(ctx, S.medium, nm * 12));
    DT_TRY(dev_alloc(ctx, S.heavy, nh * 12));
    // time slices of the window index: span >> cell_shift < kSlices
    S.cell_shift = 0;
    while (S.cell_shift < 62 && (g->span >> S.cell_shift) >= (int64_t)kSlices) ++S.cell_shift;
    DevMem ubkt2, ustart, lcell, mcell, crec;
    DT_TRY(dev_alloc(ctx, lcell, S.n_light * 2));
    DT_TRY(dev_alloc(ctx, mcell, nm * 2));
    DT_TRY(dev_alloc(ctx, crec, nc * sizeof(uint4)));
    // unit records ordered by t1 bucket (a stable two-pass radix sort on the 16-bit bucket) on the
    // first side stream, while this stream builds the other lists; the host keeps the bucket starts
    // (read back through the pinned staging buffer from byte kStageUnit; the cell starts, level
    // tables and other read-backs use the bytes before it)
    constexpr size_t kStageUnit = 32768;
    static_assert((2 * (kCells + 1) + 5 * (kLevels + 1)) * 8 <= kStageUnit, "staging layout");
    if (kStageUnit + (nbk + 1) * 4 > kPinnedStage) return fail(DT_EDEVICE, "unit bucket index exceeds staging");
    DevMem usort_tmp;
    const hipStream_t us = nu && ctx->side[0] ? ctx->side[0] : st;
    // an early return must not release buffers the side stream still uses
    struct Join {
        hipStream_t s, main;
        ~Join() {
            if (s != main) (void)hipStreamSynchronize(s);
        }
    } join{us, st};
    // (its blocks come from the cache, whose released blocks the context's stream may still use: it was idle
    // when the classes were read, and nothing is released between that and this)
    auto unit_sort = [&]() -> int {
        if (!nu) return DT_OK;
        DT_TRY(dev_alloc(ctx, ubkt2, nu * 2));
        DT_TRY(dev_alloc(ctx, S.unit, nu * sizeof(uint4)));
        DT_TRY(dev_alloc(ctx, ustart, (nbk + 1) * 4));
        DT_TRY(sort_pairs_u16_u4(ctx, ubkt.as<uint16_t>(), ubkt2.as<uint16_t>(), urec.as<uint4>(), S.unit.as<uint4>(),
                                 nu, 16, us, us != st ? &usort_tmp : nullptr));
        k_unit_starts<<<grid_for(nbk + 1, kBlock), kBlock, 0, us>>>(nu, (uint32_t)nbk, ubkt2.as<uint16_t>(),
                                                                    ustart.as<uint32_t>());
        DT_HIP(hipGetLastError());
        S.unit_index.resize(nbk + 1);
        DT_HIP(hipMemcpyAsync(ctx->pinned_stage + kStageUnit, ustart.ptr, (nbk + 1) * 4, hipMemcpyDeviceToHost, us));
        return DT_OK;
    };
    S.light_cells.assign(kCells + 1, 0);
    S.mitem_cells.assign(kCells + 1, 0);
    DT_TRY(dev_alloc(ctx, S.light_w, S.n_light * 12));
    DT_TRY(dev_alloc(ctx, S.medium_w, nm * 12));
    DT_TRY(dev_alloc(ctx, S.mlev_w, nm + 1));
    DT_TRY(dev_alloc(ctx, S.hslot, (nh + 1) * 8));
    if (n_rest) {
        k_partition<<<std::min(grid_for(n_rest, kPartTile), (unsigned)ctx->num_cus * 4), kBlock, 0, st>>>(n_rest, list,
            cls.as<uint8_t>(), g->eoff.as<uint32_t>(), g->key.as<uint64_t>(), g->shift, S.cell_shift, na, nc,
            S.light.as<uint32_t>(), S.medium.as<uint32_t>(), S.heavy.as<uint32_t>(), crec.as<uint4>(),
            lcell.as<uint16_t>(), mcell.as<uint16_t>(), ctr);
        DT_HIP(hipGetLastError());
        if (nc) {
            k_crossover<<<(unsigned)std::min<uint64_t>((nc + kBlock / 64 - 1) / (kBlock / 64), (uint64_t)ctx->num_cus * 16),
                          kBlock, 0, st>>>(nc, crec.as<uint4>(), g->eoff.as<uint32_t>(), g->key.as<uint64_t>(), g->shift,
                                           g->span, R.cost_pct, ctr);
            DT_HIP(hipGetLastError());
        }
        const unsigned tiles_l = grid_for(S.n_light, kPlaceTile), tiles_a = grid_for(na, kPlaceTile),
                       tiles_c = grid_for(nc, kPlaceTile);
        if (tiles_l + tiles_a + tiles_c) {
            k_place<<<tiles_l + tiles_a + tiles_c, kBlock, 0, st>>>(S.n_light, na, nc, tiles_l, tiles_a,
                S.light.as<uint32_t>(), lcell.as<uint16_t>(), S.medium.as<uint32_t>(), mcell.as<uint16_t>(),
                crec.as<uint4>(), S.heavy.as<uint32_t>(), S.light_w.as<uint32_t>(), S.medium_w.as<uint32_t>(),
                S.mlev_w.as<uint8_t>(), ctr);
            DT_HIP(hipGetLastError());
        }
        // work items: their sizes and totals, then the items and the tables the host keeps
        DevMem sizes, bases, tiles;
        ItemArgs A{};
        A.nm = nm;
        A.nh = nh;
        A.tiles_m = grid_for(nm + 1, kItemTile);
        A.tiles_h = grid_for(nh + 1, kItemTile);
        A.eoff = g->eoff.as<uint32_t>();
        A.medium = S.medium.as<uint32_t>();
        A.medium_w = S.medium_w.as<uint32_t>();
        A.heavy = S.heavy.as<uint32_t>();
        A.tile_stride = std::max(A.tiles_m, A.tiles_h);
        DT_TRY(dev_alloc(ctx, sizes, 2 * (nm + 1 + nh + 1) * 8));
        DT_TRY(dev_alloc(ctx, bases, 2 * (nm + 1 + nh + 1) * 8));
        DT_TRY(dev_alloc(ctx, tiles, (uint64_t)kSeqs * A.tile_stride * 8));
        unsigned long long *sz = sizes.as<unsigned long long>(), *bs = bases.as<unsigned long long>();
        A.size[0] = sz;
        A.size[1] = sz + (nm + 1);
        A.size[2] = sz + 2 * (nm + 1);
        A.size[3] = sz + 2 * (nm + 1) + (nh + 1);
        A.base[0] = bs;
        A.base[1] = bs + (nm + 1);
        A.base[2] = S.hslot.as<unsigned long long>();
        A.base[3] = bs + 2 * (nm + 1);
        A.base[4] = bs + 2 * (nm + 1) + (nh + 1);
        A.tile = tiles.as<unsigned long long>();
        k_sizes<<<A.tiles_m + A.tiles_h, kBlock, 0, st>>>(A);
        DT_HIP(hipGetLastError());
        k_tile_sums<<<1, kTileBlock, 0, st>>>(A, hs);
        DT_HIP(hipGetLastError());
        DT_TRY(unit_sort());
        DT_HIP(hipStreamSynchronize(st));
        if (hs[0] != hs[1]) return fail(DT_EDEVICE, "medium work items of the two orders differ");
        const uint64_t most_items = hs[kSeqs];
        S.n_mitems = hs[0];
        S.n_slots = hs[2];
        S.n_chunks = hs[3];
        S.n_pchunks = hs[4];
        if (S.n_chunks > 0xffffffffull || S.n_pchunks > 0xffffffffull || nh > 0xffffffffull)
            return fail(DT_EOVERFLOW, "too many heavy work items (%llu)", (unsigned long long)S.n_chunks);
        cls.reset();
        crec.reset();
        DT_TRY(dev_alloc(ctx, S.mitems, S.n_mitems * 8));
        DT_TRY(dev_alloc(ctx, S.mitems_w, S.n_mitems * 8));
        DT_TRY(dev_alloc(ctx, S.chunks, S.n_chunks * 8));
        DT_TRY(dev_alloc(ctx, S.pchunks, S.n_pchunks * 8));
        A.mitems = S.mitems.as<uint32_t>();
        A.mitems_w = S.mitems_w.as<uint32_t>();
        A.chunks = S.chunks.as<uint32_t>();
        A.pchunks = S.pchunks.as<uint32_t>();
        // workgroups a tile: about kItemsPerBlock items each, while these are no more than the chip takes
        const unsigned tiles_all = A.tiles_m + A.tiles_h, room = (unsigned)ctx->num_cus * 16;
        const unsigned share = (unsigned)std::min<uint64_t>(most_items / kItemsPerBlock, room / tiles_all);
        k_expand<<<dim3(tiles_all, std::max(share, 1u)), kBlock, 0, st>>>(A);
        DT_HIP(hipGetLastError());
        k_tables<<<1, kBlock, 0, st>>>(S.n_light, na, A, ctr, hs);
        DT_HIP(hipGetLastError());
        DT_HIP(hipStreamSynchronize(st));
        memcpy(S.light_cells.data(), hs, (kCells + 1) * 8);
        memcpy(S.mitem_cells.data(), hs + (kCells + 1), (kCells + 1) * 8);
        const unsigned long long *lt = hs + 2 * (kCells + 1);
        for (uint32_t l = 1; l <= kLevels; ++l) {
            S.med_item_at[l] = lt[0 * (kLevels + 1) + l];
            S.heavy_tri_at[l] = lt[1 * (kLevels + 1) + l];
            S.heavy_chunk_at[l] = lt[2 * (kLevels + 1) + l];
            S.heavy_pchunk_at[l] = lt[3 * (kLevels + 1) + l];
            S.heavy_slot_at[l] = lt[4 * (kLevels + 1) + l];
        }
    } else {
        DT_TRY(unit_sort());
        for (DevMem *m : {&S.mitems, &S.mitems_w, &S.chunks, &S.pchunks}) DT_TRY(dev_alloc(ctx, *m, 0));
    }
    // join the unit-record sort
    DT_HIP(hipStreamSynchronize(us));
    if (nu) memcpy(S.unit_index.data(), ctx->pinned_stage + kStageUnit, (nbk + 1) * 4);
    return DT_OK;
}

}  // namespace

// A build makes the unit keys beside its enumeration; a schedule made again makes them first.
void unit_keys(dt_graph *g, hipStream_t st) {
    k_unit_keys<<<grid_for(g->m_s, kBlock), kBlock, 0, st>>>(g->m_s, g->eoff.as<uint32_t>(), g->key.as<uint64_t>(),
                                                             g->ukey.as<uint64_t>());
}

// Where memory is short the attempt is made again with counted sizes and, if tri is needed again
// (the trials of the split), at last without unit records: those are counted on the other paths.
int make_schedule(dt_graph *g, DevMem &tri, bool last, bool with_units) {
    int rc = try_schedule(g, tri, with_units, last, false);
    if (rc == DT_ENOMEM && with_units) {
        clear_error();
        rc = try_schedule(g, tri, true, last, true);
    }
    if (rc == DT_ENOMEM && with_units && !last) {
        clear_error();
        rc = try_schedule(g, tri, false, last, true);
    }
    if (rc != DT_OK) g->sched = Schedule();
    if (rc != DT_OK || last) g->ukey.reset();
    return rc;
}

void cell_ranges(const std::vector<uint64_t> &ix, int cell_shift, const DQuery &q, Ranges &r) {
    r.n = 0;
    r.pre[0] = 0;
    if (ix.size() != kCells + 1 || ix[kCells] == 0) return;
    auto add = [&](uint64_t b, uint64_t e) {
        if (e <= b) return;
        if (r.n && r.b[r.n - 1] + (r.pre[r.n] - r.pre[r.n - 1]) == b) {
            r.pre[r.n] += e - b;   // adjacent to the previous range
            return;
        }
        r.b[r.n] = b;
        r.pre[r.n + 1] = r.pre[r.n] + (e - b);
        ++r.n;
    };
    if (!q.windowed) {
        add(0, ix[kCells]);
        return;
    }
    // relative times [wlo, whi) of the window; cells (f, l) with f <= slice(whi - 1), l >= slice(wlo)
    const uint64_t wlo = q.klo >> q.shift, whi = q.khi >> q.shift;
    if (whi <= wlo) return;
    const uint64_t ql = std::min<uint64_t>(wlo >> cell_shift, kSlices - 1);
    const uint64_t qh = std::min<uint64_t>((whi - 1) >> cell_shift, kSlices - 1);
    for (uint64_t f = 0; f <= qh; ++f) add(ix[f * kSlices + ql], ix[f * kSlices + kSlices]);
}

void unit_range(const dt_graph *g, const DQuery &q, uint64_t *b, uint64_t *e) {
    const Schedule &S = g->sched;
    *b = 0;
    *e = S.n_unit;
    if (!q.windowed || S.n_unit == 0) return;
    // a triangle inside the window has wlo <= t1 < whi (relative times): buckets
    // wlo >> shift .. (whi - 1) >> shift
    const std::vector<uint32_t> &ix = S.unit_index;   // bucket starts, nbk + 1 entries
    const uint64_t nbk = ix.size() - 1;
    const uint64_t wlo = q.klo >> q.shift, whi = q.khi >> q.shift;
    if (whi <= wlo) {
        *e = *b;
        return;
    }
    const uint64_t bl = std::min<uint64_t>(wlo >> S.unit_shift, nbk);
    const uint64_t bh = std::min<uint64_t>(((whi - 1) >> S.unit_shift) + 1, nbk);
    *b = ix[bl];
    *e = bh > bl ? ix[bh] : ix[bl];
}

}  // namespace dt
