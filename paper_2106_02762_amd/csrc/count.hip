// Per-triangle temporal counting (Algorithm 4 with Algorithms 1-3, Section 5 and Appendix A) and
// the per-type reduction.
//
// Every static triangle <u, v, w> (u first in the degeneracy ordering, v before w) owns six
// key-sorted edge lists: uv+ (u->v), uv- (v->u), uw+, uw-, vw+, vw-.  A cell (pi, rho) of the
// paper is an ordering pi (Figure 3) and one direction per pair rho (Figure 4); its count goes to
// type psi(pi, rho) (Table 2).  Only the lists on the two pairs at u are ever walked; the {v,w}
// lists are only searched (Section 5, "source vertex").
//
// Paths, chosen per triangle by the scheduler:
//  - unit: a triangle with one temporal edge on each pair has its ordering, orientation and type
//    fixed at build time; a query tests the record's three times against its deltas and window
//    (Definition 1) and adds one to that type.  A pure stream of 16-byte records.
//  - light: one lane walks every pair (x, y) of edges from the uv and uw lists (the pairwise form
//    of Lemma 1).  With x, y fixed and ordered, the third edge z on {v,w} is first, middle or last,
//    and each case is one key range of the vw list found by binary search; that is cells
//    (pi5|pi6), (pi3|pi4) and (pi1|pi2) respectively.
//  - medium: one lane per edge x of the triangle's smaller source-incident pair; only the edges y
//    of the other pair within d13 of x can complete a triangle, so the lane finds those by binary
//    search, and each wavefront spreads the (x, y) pairs of its lanes evenly over them, each pair
//    then handled as on the light path.
//  - heavy: the prefix-count procedures.  For every edge on a uv or uw list a prefix pass stores
//    the cumulative counts that Algorithms 1-3 need (CEC of Section 5), and a second pass walks
//    the same edges as e2 (Algorithm 1: pi1/pi2), e1 (Algorithm 2: pi3/pi4) and e2 (Algorithm 3:
//    pi5/pi6), each with a constant number of binary searches, split into chunks across
//    workgroups.  The formulas are the paper's, restated for keys (t, input index) so that equal
//    timestamps are handled, with the region bounds written as max/min clamps.
//
// A query with a time window walks the windowed copies of the light and medium lists, ordered by
// window cell, and only the cells that can hold a triangle inside its window (the unit records by
// their first time likewise).
//
// Counts are int64 and summed per lane, per wave, per block, then per launch, with no atomics on
// the result (cells mode, a diagnostic, uses atomics).
#include <type_traits>

#include "count_dev.h"

namespace dt {

using namespace cdev;

namespace {

// ACC: Acc<false> (int64 type counts), Acc<true> (the 48 cells by atomics, no partials) or AccW
// (128-bit type counts, 16-word partial slots)
template <class ACC> constexpr bool kCellsAcc = std::is_same<ACC, Acc<true>>::value;
template <class ACC> constexpr int kAccWords = std::is_same<ACC, AccW>::value ? 2 : 1;

// body(accumulator) of a pairwise kernel with accumulator ACC, then its block's partial slot
template <class ACC, unsigned BLOCK, class BODY>
__device__ __forceinline__ void with_pairwise(int64_t *__restrict__ partial, int64_t *__restrict__ cells, BODY &&body) {
    if constexpr (kCellsAcc<ACC>) {
        AccCells acc{cells};
        body(acc);
    } else {
        __shared__ unsigned long long s_col[8 * kAccWords<ACC> * BLOCK];
        AccLane<BLOCK, kAccWords<ACC>> acc(s_col);
        body(acc);
        ACC out;
        acc.get(out.t);
        acc_store<BLOCK>(out, partial, blockIdx.x);
    }
}

// light path: block b of nblk takes a contiguous run of the list's ranges
template <unsigned BLOCK, class PACC>
__device__ __forceinline__ void light_block(uint32_t b, uint32_t nblk, const Ranges &R, const uint32_t *__restrict__ tri,
                                            const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key,
                                            const DQuery &q, PACC &acc) {
    const uint64_t n_tri = R.pre[R.n];
    const uint64_t per = (n_tri + nblk - 1) / nblk;
    const uint64_t beg = (uint64_t)xcd_block(b, nblk) * per;
    const uint64_t end = beg + per < n_tri ? beg + per : n_tri;
    uint32_t r = 0;
    for (uint64_t i = beg + threadIdx.x; i < end; i += BLOCK) {
        const uint64_t t = range_at(R, r, i);
        light_tri(tri[3 * t], tri[3 * t + 1], tri[3 * t + 2], eoff, key, q, acc);
    }
}

// medium path: wave w takes the 64 entries from 64 w on, then those from 64 (w + W) on, ...;
// with lev (windowed copies) entries of triangles below the query's level are skipped
template <unsigned BLOCK, class PACC>
__device__ __forceinline__ void medium_block(uint32_t b, uint32_t nblk, const Ranges &R, const uint32_t *__restrict__ med,
                                             const uint32_t *__restrict__ ent, const uint8_t *__restrict__ lev,
                                             const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key,
                                             const DQuery &q, PACC &acc) {
    const unsigned lane = threadIdx.x & 63;
    const uint64_t n_ent = R.pre[R.n];
    const uint64_t W = (uint64_t)nblk * (BLOCK / 64);
    uint32_t r = 0;
    for (uint64_t e = ((uint64_t)b * (BLOCK / 64) + threadIdx.x / 64) * 64; e < n_ent; e += W * 64) {
        const uint64_t j = e + lane;
        const bool active = j < n_ent;
        // one visit per outer edge, plus the wavefront's close pairs (counted by lane 0)
        const uint32_t pairs = medium_lanes(med, ent, active ? range_at(R, r, j) : 0, active, eoff, key, q, acc, lane, lev);
        acc.visits += (active ? 1u : 0u) + (lane == 0 ? pairs : 0u);
    }
}

// The same with the pairs of the wavefronts' largest groups of 64 entries shared by the block: at large
// deltas a group holds up to a hundred thousand pairs where the mean is ten thousand, and the last
// wavefronts ran alone for most of the kernel (61M edges without deltas: count 2.4 -> 1.7 ms; 100K edges
// 0.36 -> 0.16).  A wavefront keeps the largest group of more than kShareMin pairs that
// it meets for the end, in LDS; the block then evaluates its kept groups together.  Consecutive groups,
// which often are of one large triangle, go to different blocks.
constexpr uint32_t kShareMin = 512;
constexpr unsigned kShareWords = 10;
template <unsigned BLOCK, class PACC>
__device__ __forceinline__ void medium_shared(uint32_t b, uint32_t nblk, const Ranges &R, const uint32_t *__restrict__ med,
                                              const uint32_t *__restrict__ ent, const uint8_t *__restrict__ lev,
                                              const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key,
                                              const DQuery &q, PACC &acc) {
    constexpr unsigned kWaves = BLOCK / 64;
    __shared__ uint32_t s_kept[kWaves][kShareWords][64];
    __shared__ uint32_t s_total[kWaves];
    const unsigned lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    auto keep = [&](const MediumLanes &M) {
        const uint32_t w[kShareWords] = {M.excl, M.c0, M.lo0, M.lo1, M.flags, M.kx_lo, M.kx_hi, M.z0, M.z1, M.z2};
#pragma unroll
        for (unsigned x = 0; x < kShareWords; ++x) s_kept[wave][x][lane] = w[x];
    };
    auto kept = [&](unsigned g, uint32_t total) {
        uint32_t w[kShareWords];
#pragma unroll
        for (unsigned x = 0; x < kShareWords; ++x) w[x] = s_kept[g][x][lane];
        return MediumLanes{w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7], w[8], w[9], total};
    };
    auto eval = [&](uint32_t d_uv, uint32_t d_uw, uint32_t z0, uint32_t z1, uint32_t z2, uint64_t k_uv, uint64_t k_uw) {
        pair_thirds(key, z0, z1, z2, q, d_uv, d_uw, k_uv, k_uw, acc);
    };
    const uint64_t n_ent = R.pre[R.n];
    const uint64_t W = (uint64_t)nblk * kWaves;
    uint32_t r = 0, held = 0;
    for (uint64_t e = ((uint64_t)wave * nblk + b) * 64; e < n_ent; e += W * 64) {
        const uint64_t j = e + lane;
        const bool active = j < n_ent;
        MediumLanes M = medium_find(med, ent, active ? range_at(R, r, j) : 0, active, eoff, key, q, lane, lev);
        acc.visits += (active ? 1u : 0u) + (lane == 0 ? M.total : 0u);
        if (M.total > kShareMin && M.total > held) {
            const MediumLanes old = kept(wave, held);
            keep(M);
            held = M.total;
            M = old;
        }
        medium_spread(M, 0, 64, key, eval, lane);
    }
    if (lane == 0) s_total[wave] = held;
    __syncthreads();
    for (unsigned g = 0; g < kWaves; ++g) {
        const uint32_t total = s_total[g];
        if (total) medium_spread(kept(g, total), wave * 64, BLOCK, key, eval, lane);
    }
}

// unit path: block b of nblk takes a contiguous run of the records [beg, end); returns its length
template <bool CELLS, unsigned BLOCK>
__device__ __forceinline__ uint64_t unit_block(uint32_t b, uint32_t nblk, uint64_t beg, uint64_t end,
                                               const uint4 *__restrict__ rec, const UQuery &u, uint32_t (&c)[8],
                                               int64_t *__restrict__ cells) {
    const uint64_t per = (end - beg + nblk - 1) / nblk;
    const uint64_t rb = beg + (uint64_t)b * per;
    const uint64_t re = rb + per < end ? rb + per : end;
    if (rb >= re) return 0;
    unit_run<CELLS, BLOCK>(rec, rb, re, u, c, cells);
    return re - rb;
}

template <class ACC, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_light(Ranges R, const uint32_t *__restrict__ tri, const uint32_t *__restrict__ eoff,
        const uint64_t *__restrict__ key, DQuery q, int64_t *__restrict__ partial,
        int64_t *__restrict__ cells, unsigned long long *__restrict__ visits) {
    with_pairwise<ACC, BLOCK>(partial, cells, [&](auto &acc) {
        light_block<BLOCK>(blockIdx.x, gridDim.x, R, tri, eoff, key, q, acc);
        add_visits(visits, acc.visits);
    });
}

// (the shared form has at most as many blocks as partial slots, and at least half as many: its blocks
// zero the others)
template <unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_medium_shared(Ranges R, const uint32_t *__restrict__ med, const uint32_t *__restrict__ ent,
                const uint8_t *__restrict__ lev, const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key,
                DQuery q, int64_t *__restrict__ partial, unsigned slots, unsigned long long *__restrict__ visits) {
    with_pairwise<Acc<false>, BLOCK>(partial, nullptr, [&](auto &acc) {
        medium_shared<BLOCK>(blockIdx.x, gridDim.x, R, med, ent, lev, eoff, key, q, acc);
        add_visits(visits, acc.visits);
    });
    if (threadIdx.x < 8 && gridDim.x + blockIdx.x < slots) partial[8 * (uint64_t)(gridDim.x + blockIdx.x) + threadIdx.x] = 0;
}

template <class ACC, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_medium(Ranges R, const uint32_t *__restrict__ med, const uint32_t *__restrict__ ent,
         const uint8_t *__restrict__ lev, const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key,
         DQuery q, int64_t *__restrict__ partial, int64_t *__restrict__ cells, unsigned long long *__restrict__ visits) {
    with_pairwise<ACC, BLOCK>(partial, cells, [&](auto &acc) {
        medium_block<BLOCK>(blockIdx.x, gridDim.x, R, med, ent, lev, eoff, key, q, acc);
        add_visits(visits, acc.visits);
    });
}

template <class ACC, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_unit(uint64_t beg, uint64_t end, const uint4 *__restrict__ rec, UQuery u, int64_t *__restrict__ partial,
       int64_t *__restrict__ cells, unsigned long long *__restrict__ visits) {
    uint32_t c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const uint64_t n = unit_block<kCellsAcc<ACC>, BLOCK>(blockIdx.x, gridDim.x, beg, end, rec, u, c, cells);
    if (visits && threadIdx.x == 0 && n) atomicAdd(visits, (unsigned long long)n);
    if (!kCellsAcc<ACC>) {
        ACC acc;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc.t[j] = c[j];
        acc_store<BLOCK>(acc, partial, blockIdx.x);
    }
}

// The three paths of one count in one launch: mg medium blocks (the longest chains first), then lg light
// ones and ug unit ones, each with its own partial slot.
struct SmallCount {
    Ranges lr, mr;
    const uint32_t *light, *medium, *mitems, *eoff;
    const uint8_t *mlev;
    const uint64_t *key;
    const uint4 *unit;
    uint64_t ub, ue;
    DQuery q;
    UQuery u;
    uint32_t mg, lg, ug;
};
template <class ACC, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_small(SmallCount C, int64_t *__restrict__ partial) {
    const uint32_t b = blockIdx.x;
    if (b >= C.mg + C.lg) {
        uint32_t c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        unit_block<false, BLOCK>(b - C.mg - C.lg, C.ug, C.ub, C.ue, C.unit, C.u, c, nullptr);
        ACC acc;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc.t[j] = c[j];
        acc_store<BLOCK>(acc, partial, b);
        return;
    }
    with_pairwise<ACC, BLOCK>(partial, nullptr, [&](auto &acc) {
        if (b < C.mg) medium_shared<BLOCK>(b, C.mg, C.mr, C.medium, C.mitems, C.mlev, C.eoff, C.key, C.q, acc);
        else light_block<BLOCK>(b - C.mg, C.lg, C.lr, C.light, C.eoff, C.key, C.q, acc);
    });
}

// ---------------------------------------------------------------------------------------------
// heavy path (the per-item bodies are in count_dev.h, shared with the batched kernel)
// ---------------------------------------------------------------------------------------------
// The heavy work of up to kSweepMax queries over the same triangles, each with its own scratch: block
// row y of every kernel is query y.
struct HeavySet {
    HeavyArgs A[kSweepMax];
};

// window-clipped bounds of the six lists of every heavy triangle of the query
__global__ void k_heavy_clip(HeavySet S, uint64_t n_q) {
    const uint64_t h = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (h < n_q) heavy_clip_one(S.A[blockIdx.y], h);
}

// phase 1 of the prefix pass over prefix chunks [A.pb, pe)
__global__ void __launch_bounds__(kPrefixBlock)
k_heavy_prefix_local(HeavySet S, uint64_t pe, unsigned long long *__restrict__ visits) {
    const HeavyArgs &A = S.A[blockIdx.y];
    uint64_t vis = 0;
    for (uint64_t c = A.pb + blockIdx.x; c < pe; c += gridDim.x) heavy_prefix_local_chunk(A, c, vis);
    add_visits(visits, vis);
}

// phase 2: the carries between the chunks of each list (a thread per chunk, the list's first works)
__global__ void k_heavy_prefix_scan(HeavySet S, uint64_t pe) {
    const HeavyArgs &A = S.A[blockIdx.y];
    const uint64_t c = A.pb + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < pe) heavy_prefix_scan_list(A, c, pe);
}

// phase 3: every chunk adds its carry
__global__ void __launch_bounds__(kPrefixBlock)
k_heavy_prefix_add(HeavySet S, uint64_t pe) {
    const HeavyArgs &A = S.A[blockIdx.y];
    for (uint64_t c = A.pb + blockIdx.x; c < pe; c += gridDim.x) heavy_prefix_add_chunk(A, c);
}

// the count pass: chunks [cb, ce) of 256 source edges (of the four lists in a row) each
template <class ACC, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_heavy_count(HeavySet S, uint64_t cb, uint64_t ce, int64_t *__restrict__ partial, int64_t *__restrict__ cells,
              unsigned long long *__restrict__ visits) {
    const HeavyArgs &A = S.A[blockIdx.y];
    ACC acc;
    acc.cells = cells;
    for (uint64_t ch = cb + blockIdx.x; ch < ce; ch += gridDim.x) heavy_count_chunk(A, ch, acc);
    add_visits(visits, acc.visits);
    if (!kCellsAcc<ACC>) acc_store<BLOCK>(acc, partial, (uint64_t)blockIdx.y * gridDim.x + blockIdx.x);
}

// final reduction of the per-block partials into out8 (deterministic order)
// (thread i adds word i, i + 1024, ... of the partials, all of type i % 8: 8192 slots 22 -> 8 us against
// a slot per thread and 256 threads)
constexpr unsigned kReduceBlock = 1024;
__device__ __forceinline__ void reduce_words(uint64_t n_words, const int64_t *__restrict__ partial, int64_t &t) {
    uint64_t i = threadIdx.x;
    for (; i + 3 * kReduceBlock < n_words; i += 4 * kReduceBlock) {
        const int64_t a = partial[i], b = partial[i + kReduceBlock], c = partial[i + 2 * kReduceBlock],
                      d = partial[i + 3 * kReduceBlock];
        t += a + b + c + d;
    }
    for (; i < n_words; i += kReduceBlock) t += partial[i];
}
// thread i's sum t (of type i % 8) over the block into out8
__device__ __forceinline__ void reduce_store(int64_t t, int64_t *__restrict__ out8) {
    __shared__ int64_t s[kReduceBlock / 64][8];
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) t += __shfl_xor((long long)t, o, 64);
    if ((threadIdx.x & 63) < 8) s[threadIdx.x / 64][threadIdx.x & 7] = t;
    __syncthreads();
    if (threadIdx.x < 8) {
        int64_t v = 0;
#pragma unroll
        for (unsigned w = 0; w < kReduceBlock / 64; ++w) v += s[w][threadIdx.x];
        out8[threadIdx.x] = v;
    }
}
__global__ void __launch_bounds__(kReduceBlock)
k_reduce(uint64_t n_part, const int64_t *__restrict__ partial, int64_t *__restrict__ out8) {
    int64_t t = 0;
    reduce_words(8 * n_part, partial, t);
    reduce_store(t, out8);
}

// the 128-bit form: 16-word partials into 16 words (low, high per type)
__global__ void __launch_bounds__(256)
k_reduce_w(uint64_t n_part, const int64_t *__restrict__ partial, int64_t *__restrict__ out16) {
    AccW acc;
    for (uint64_t i = threadIdx.x; i < n_part; i += 256) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            acc.t[j] += ((unsigned __int128)(uint64_t)partial[16 * i + 2 * j + 1] << 64) | (uint64_t)partial[16 * i + 2 * j];
    }
    block_store_w<256>(acc.t, out16);
}

__global__ void k_zero(uint64_t n, int64_t *__restrict__ p) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------------------------------------
// sweeps: several delta triples (one window) per visit of the triangle data
// ---------------------------------------------------------------------------------------------
struct SweepQ {
    DQuery q[kSweepMax];
    UQuery u[kSweepMax];
    uint32_t k;
    int64_t d13max;   // largest d13 of the k triples
    uint32_t qlev;    // its level: the pass's medium / heavy split
};

// one (uv edge, uw edge) pair against every triple
__device__ __forceinline__ void sweep_pair(const uint64_t *__restrict__ key, uint32_t z0, uint32_t z1, uint32_t z2,
                                           const SweepQ &Q, uint32_t d_uv, uint32_t d_uw, uint64_t k_uv, uint64_t k_uw,
                                           unsigned long long *sw) {
    const int64_t t_uv = (int64_t)(k_uv >> Q.q[0].shift), t_uw = (int64_t)(k_uw >> Q.q[0].shift);
    if ((t_uv < t_uw ? t_uw - t_uv : t_uv - t_uw) > Q.d13max) return;
    for (uint32_t j = 0; j < Q.k; ++j) {
        AccShared a{sw + 8 * j};
        pair_thirds(key, z0, z1, z2, Q.q[j], d_uv, d_uw, k_uv, k_uw, a);
    }
}

// a block's sweep counters (per wavefront, [8 j + type]) to its partial slots
template <unsigned BLOCK>
__device__ __forceinline__ void sweep_flush(unsigned long long (*s_sw)[kSweepMax * 8], uint32_t k,
                                            int64_t *__restrict__ part, uint64_t slot) {
    __syncthreads();
    if (threadIdx.x < 8 * k) {
        unsigned long long v = 0;
#pragma unroll
        for (unsigned w = 0; w < BLOCK / 64; ++w) v += s_sw[w][threadIdx.x];
        part[8 * (slot * k + threadIdx.x / 8) + threadIdx.x % 8] = (int64_t)v;
    }
}

// unit records: each record is read once and tested against every delta triple.  A wavefront
// takes 64 records at a time; for each triple the lanes' pass/fail bits form one 64-bit ballot, as
// do the lanes of each type.  Lane l keeps the wavefront's count of (triple l / 8, type l % 8): it
// adds the popcount of that triple's ballot masked by that type's ballot.
template <unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_unit_sweep(uint64_t beg, uint64_t end, const uint4 *__restrict__ rec, SweepQ Q, int64_t *__restrict__ part,
             uint64_t slot0) {
    static_assert(kSweepMax * 8 == 64, "one counter per lane");
    __shared__ uint32_t s_cnt[BLOCK / 64][64];
    const unsigned lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    const uint32_t my_j = lane >> 3, my_t = lane & 7;
    const uint64_t n = end - beg;
    const uint64_t per = (n + gridDim.x - 1) / gridDim.x;
    const uint64_t b = beg + (uint64_t)blockIdx.x * per;
    const uint64_t e = b + per < end ? b + per : end;
    uint32_t cnt = 0;
    // the window is the same for every triple: test it once per record
    const uint32_t wlo = Q.u[0].wlo, whi = Q.u[0].whi;
    auto test = [&](const uint4 r, bool valid) {
        const uint32_t g13 = r.y + r.z, ty = r.w & 7u;
        valid = valid && r.x >= wlo && r.x + g13 < whi;
        uint64_t tsel = 0, jsel = 0;
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t) {
            const uint64_t m = __ballot(valid && ty == t);
            tsel = my_t == t ? m : tsel;
        }
#pragma unroll
        for (uint32_t j = 0; j < kSweepMax; ++j) {
            if (j < Q.k) {
                const UQuery &u = Q.u[j];
                const uint64_t m = __ballot(valid && r.y <= u.d12 && r.z <= u.d23 && g13 <= u.d13);
                jsel = my_j == j ? m : jsel;
            }
        }
        cnt += (uint32_t)__popcll(jsel & tsel);
    };
    // two records per lane in flight; the loop bounds are the same for the whole wavefront
    uint64_t base = b + 64 * wave;
    for (; base + BLOCK < e; base += 2 * BLOCK) {
        const uint64_t i0 = base + lane, i1 = base + BLOCK + lane;
        const bool v1 = i1 < e;
        const uint4 r0 = rec[i0];
        const uint4 r1 = v1 ? rec[i1] : make_uint4(0u, 0u, 0u, 0u);
        test(r0, true);
        test(r1, v1);
    }
    if (base < e) {
        const uint64_t i0 = base + lane;
        const bool v0 = i0 < e;
        test(v0 ? rec[i0] : make_uint4(0u, 0u, 0u, 0u), v0);
    }
    s_cnt[wave][lane] = cnt;
    __syncthreads();
    if (threadIdx.x < 8 * Q.k) {
        int64_t v = 0;
#pragma unroll
        for (unsigned w = 0; w < BLOCK / 64; ++w) v += s_cnt[w][threadIdx.x];
        part[8 * ((slot0 + blockIdx.x) * Q.k + threadIdx.x / 8) + threadIdx.x % 8] = v;
    }
}

// light triangles: each lane's triangles once, every pair tested against every triple
template <unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_light_sweep(Ranges R, const uint32_t *__restrict__ tri, const uint32_t *__restrict__ eoff,
              const uint64_t *__restrict__ key, SweepQ Q, int64_t *__restrict__ part, uint64_t slot0) {
    __shared__ unsigned long long s_sw[BLOCK / 64][kSweepMax * 8];
    for (unsigned x = threadIdx.x; x < (BLOCK / 64) * kSweepMax * 8; x += BLOCK) (&s_sw[0][0])[x] = 0;
    __syncthreads();
    unsigned long long *sw = s_sw[threadIdx.x / 64];
    const uint64_t n_tri = R.pre[R.n];
    const uint32_t nblk = gridDim.x;
    const uint32_t b = xcd_block(blockIdx.x, nblk);
    const uint64_t per = (n_tri + nblk - 1) / nblk;
    const uint64_t beg = (uint64_t)b * per;
    const uint64_t end = beg + per < n_tri ? beg + per : n_tri;
    uint32_t r = 0;
    for (uint64_t i = beg + threadIdx.x; i < end; i += BLOCK) {
        const uint64_t t = range_at(R, r, i);
        const uint32_t e_vw = tri[3 * t + 2];
        const uint32_t z0 = eoff[2 * e_vw], z1 = eoff[2 * e_vw + 1], z2 = eoff[2 * e_vw + 2];
        // (one window for all)
        light_pairs(eoff, tri[3 * t], tri[3 * t + 1], key, Q.q[0],
                    [&](uint32_t d_uv, uint32_t d_uw, uint64_t k_uv, uint64_t k_uw) {
                        sweep_pair(key, z0, z1, z2, Q, d_uv, d_uw, k_uv, k_uw, sw);
                    });
    }
    sweep_flush<BLOCK>(s_sw, Q.k, part, slot0 + blockIdx.x);
}

// medium entries: each entry's close pairs found once, for the largest d13 of the triples, and
// every pair tested against every triple
template <unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK)
k_medium_sweep(Ranges R, const uint32_t *__restrict__ med, const uint32_t *__restrict__ ent,
               const uint8_t *__restrict__ lev, const uint32_t *__restrict__ eoff, const uint64_t *__restrict__ key, SweepQ Q,
               int64_t *__restrict__ part, uint64_t slot0) {
    __shared__ unsigned long long s_sw[BLOCK / 64][kSweepMax * 8];
    for (unsigned x = threadIdx.x; x < (BLOCK / 64) * kSweepMax * 8; x += BLOCK) (&s_sw[0][0])[x] = 0;
    __syncthreads();
    unsigned long long *sw = s_sw[threadIdx.x / 64];
    const unsigned lane = threadIdx.x & 63;
    const uint64_t n_ent = R.pre[R.n];
    const uint64_t W = (uint64_t)gridDim.x * (BLOCK / 64);
    DQuery qr = Q.q[0];   // the window, the widest closeness and the pass's medium / heavy split
    qr.d13 = Q.d13max;
    qr.qlev = Q.qlev;
    uint32_t r = 0;
    for (uint64_t b = ((uint64_t)blockIdx.x * (BLOCK / 64) + threadIdx.x / 64) * 64; b < n_ent; b += W * 64) {
        const uint64_t x = b + lane;
        const bool active = x < n_ent;
        medium_lanes_eval(med, ent, active ? range_at(R, r, x) : 0, active, eoff, key, qr,
                          [&](uint32_t d_uv, uint32_t d_uw, uint32_t z0, uint32_t z1, uint32_t z2, uint64_t k_uv,
                              uint64_t k_uw) { sweep_pair(key, z0, z1, z2, Q, d_uv, d_uw, k_uv, k_uw, sw); },
                          lane, lev);
    }
    sweep_flush<BLOCK>(s_sw, Q.k, part, slot0 + blockIdx.x);
}

// out[8 j + i] = sum over slots of part[8 (K slot + j) + i] and over x of heavy[8 (n_heavy j + x) + i];
// block j for query j
__global__ void __launch_bounds__(kReduceBlock)
k_reduce_sweep(uint64_t n_slot, uint32_t k, const int64_t *__restrict__ part, uint64_t n_heavy,
               const int64_t *__restrict__ heavy, int64_t *__restrict__ out) {
    const uint32_t j = blockIdx.x;
    int64_t t = 0;
    if (n_heavy) reduce_words(8 * n_heavy, heavy + 8 * n_heavy * j, t);
#pragma unroll 4
    for (uint64_t i = threadIdx.x / 8; i < n_slot; i += kReduceBlock / 8) t += part[8 * (i * k + j) + (threadIdx.x & 7)];
    reduce_store(t, out + 8 * j);
}

constexpr unsigned kLightBlock = 256;
constexpr unsigned kUnitBlock = 256;
constexpr uint64_t kUnitPerBlock = 16384;   // records per workgroup at least (64 per thread)
// Counts of up to this many light, medium and unit blocks per CU take them in one launch: they are all
// resident at once, so the three kernels side by side would overlap no more, and the fork, the two joins
// and two launches cost more than the work (10K edges: 72 -> 31 us).  Larger counts fork, where
// each kernel's own registers leave more wavefronts in flight.
constexpr unsigned kSmallPerCu = 4;
constexpr uint64_t kSweepHeavyBytes = 1ull << 30;   // prefix arrays of a sweep's queries at a time

}  // namespace

int normalise_query(const dt_graph *g, const dt_query *qq, DQuery *out, bool *empty) {
    if (!qq) return fail(DT_EINVAL, "null query");
    if (qq->d13 < 0 || qq->d12 < 0 || qq->d23 < 0)
        return fail(DT_EINVAL, "deltas must be >= 0 (got %lld, %lld, %lld)", (long long)qq->d13,
                    (long long)qq->d12, (long long)qq->d23);
    if (qq->t_lo > qq->t_hi) return fail(DT_EINVAL, "window t_lo > t_hi");
    DQuery q{};
    const int64_t span = g->span;
    auto clampd = [&](int64_t d) { return d > span ? span : d; };
    int64_t d13 = clampd(qq->d13), d12 = clampd(qq->d12), d23 = clampd(qq->d23);
    // the same constraint set: t2-t1 <= t3-t1 and t3-t2 <= t3-t1, and t3-t1 = (t3-t2)+(t2-t1)
    d12 = d12 < d13 ? d12 : d13;
    d23 = d23 < d13 ? d23 : d13;
    d13 = d13 < d12 + d23 ? d13 : d12 + d23;
    q.d13 = d13;
    q.d12 = d12;
    q.d23 = d23;
    q.qlev = query_level(d13);
    q.span = span;
    q.shift = g->shift;
    *empty = (g->m == 0);
    if (qq->t_lo <= g->t_min && qq->t_hi >= g->t_max) {
        q.windowed = 0;
        q.klo = 0;
        q.khi = ~0ull;
    } else {
        q.windowed = 1;
        if (qq->t_hi < g->t_min || qq->t_lo > g->t_max) {
            *empty = true;
            q.klo = q.khi = 0;
        } else {
            int64_t lo = qq->t_lo < g->t_min ? 0 : qq->t_lo - g->t_min;
            int64_t hi = qq->t_hi > g->t_max ? span : qq->t_hi - g->t_min;   // inclusive
            q.klo = (uint64_t)lo << g->shift;
            q.khi = (uint64_t)(hi + 1) << g->shift;
        }
    }
    *out = q;
    return DT_OK;
}

void medium_ranges(const dt_graph *g, const DQuery &q, Ranges &r, const uint8_t **lev) {
    const Schedule &S = g->sched;
    if (q.windowed) {
        cell_ranges(S.mitem_cells, S.cell_shift, q, r);
        *lev = S.mlev_w.as<uint8_t>();
        return;
    }
    // whole span: the entries of the always-medium triangles and of the contested ones at or above
    // the query's level, a prefix of the list
    const uint64_t e = S.med_item_at[q.qlev < kLevels ? q.qlev : kLevels];
    r.n = e ? 1 : 0;
    r.pre[0] = 0;
    if (e) {
        r.b[0] = 0;
        r.pre[1] = e;
    }
    *lev = nullptr;
}

void heavy_range(const dt_graph *g, const DQuery &q, HeavyRange &h) {
    const Schedule &S = g->sched;
    const uint32_t l = q.qlev < kLevels ? q.qlev : kLevels;
    h.hb = S.heavy_tri_at[l];
    h.cb = S.heavy_chunk_at[l];
    h.pb = S.heavy_pchunk_at[l];
    h.slot_base = S.heavy_slot_at[l];
    h.n = S.n_heavy - h.hb;
    h.scratch_bytes = h.n ? (S.n_slots - h.slot_base) * kVals * sizeof(int64_t) + 12 * 4 * h.n +
                                (S.n_pchunks - h.pb) * kVals * sizeof(int64_t) + 512
                          : 0;
}

void heavy_args(const dt_graph *g, const DQuery &q, const HeavyRange &hr, uint8_t *scratch, HeavyArgs &A) {
    const Schedule &S = g->sched;
    const uint64_t ns = S.n_slots - hr.slot_base, npc = S.n_pchunks - hr.pb;
    A.heavy = S.heavy.as<uint32_t>();
    A.pchunks = S.pchunks.as<uint32_t>();
    A.chunks = S.chunks.as<uint32_t>();
    A.eoff = g->eoff.as<uint32_t>();
    A.key = g->key.as<uint64_t>();
    A.hslot = S.hslot.as<uint64_t>();
    A.hb = hr.hb;
    A.pb = hr.pb;
    A.slot_base = hr.slot_base;
    A.ns = ns;
    A.P = reinterpret_cast<int64_t *>(scratch);
    A.T = A.P + ns * kVals;
    A.clip = reinterpret_cast<uint32_t *>(A.T + npc * kVals);
    A.q = q;
}

void count_plan(const dt_graph *g, const DQuery &q, unsigned parts, CountPlan &p) {
    const dt_ctx *ctx = g->ctx;
    const Schedule &S = g->sched;
    p.parts = parts;
    const bool do_light = parts & 1, do_medium = parts & 2, do_heavy = parts & 4;
    // the parts of the light and medium lists the query sees (window cells; the medium / heavy
    // split of its level)
    cell_ranges(S.light_cells, S.cell_shift, q, p.lr);
    medium_ranges(g, q, p.mr, &p.mlev);
    const uint64_t nl = p.lr.pre[p.lr.n], nmi = p.mr.pre[p.mr.n];
    p.light = (q.windowed ? S.light_w : S.light).as<uint32_t>();
    p.medium = (q.windowed ? S.medium_w : S.medium).as<uint32_t>();
    p.mitems = (q.windowed ? S.mitems_w : S.mitems).as<uint32_t>();
    const CountGeom &G = g->geom;
    const unsigned light_grid = (nl && do_light) ? (unsigned)std::min<uint64_t>(
        (nl + kLightBlock - 1) / kLightBlock, (uint64_t)ctx->num_cus * G.light_bpc) : 0;
    p.lg = light_grid ? ((light_grid + 7) / 8) * 8 : 0;
    heavy_range(g, q, p.hr);
    if (!do_heavy) p.hr.n = 0;
    p.hg = p.hr.n ? (unsigned)std::min<uint64_t>(S.n_chunks - p.hr.cb, (uint64_t)ctx->num_cus * 16) : 0;
    p.mg = (nmi && do_medium) ? (unsigned)std::min<uint64_t>((nmi + 255) / 256, (uint64_t)ctx->num_cus * G.medium_bpc) : 0;
    p.ub = p.ue = 0;
    if (S.n_unit && (parts & 8)) unit_range(g, q, &p.ub, &p.ue);
    p.ug = p.ue > p.ub ? (unsigned)std::min<uint64_t>((p.ue - p.ub + kUnitPerBlock - 1) / kUnitPerBlock,
                                                      (uint64_t)ctx->num_cus * 8) : 0;
    p.n_part = (uint64_t)p.lg + p.hg + p.mg + p.ug;
    // graphs whose counts may pass 2^63 are counted in 128 bits (16-word partials, 16-word result)
    p.wide = (g->sum_sigma3 >> 63) != 0;
    p.part_bytes = (p.n_part + 1) * (p.wide ? 16 : 8) * sizeof(int64_t);
    p.heavy_bytes = p.hr.n ? p.hr.scratch_bytes : 0;
}

// The heavy kernels of k queries over the range hr on stream s: scratch of query j at scratch + j *
// hr.scratch_bytes, partial slots of query j from j * hg on.
template <class ACC>
int launch_heavy(dt_graph *g, const DQuery *qs, uint32_t k, const HeavyRange &hr, unsigned hg, uint8_t *scratch,
                 int64_t *part, hipStream_t s, int64_t *cells_dev, unsigned long long *visits) {
    dt_ctx *ctx = g->ctx;
    const Schedule &S = g->sched;
    if (g->tuning.heavy_chunk != 256) return fail(DT_EINVAL, "heavy_chunk %u not compiled", g->tuning.heavy_chunk);
    HeavySet H;
    for (uint32_t j = 0; j < k; ++j) heavy_args(g, qs[j], hr, scratch + j * hr.scratch_bytes, H.A[j]);
    const uint64_t npc = S.n_pchunks - hr.pb;
    const unsigned pgrid = (unsigned)std::min<uint64_t>(npc, (uint64_t)ctx->num_cus * 16);
    k_heavy_clip<<<dim3(grid_for(hr.n, 256), k), 256, 0, s>>>(H, hr.n);
    DT_HIP(hipGetLastError());
    prof_begin(ctx, kProfHeavyPrefix, s);
    k_heavy_prefix_local<<<dim3(pgrid, k), kPrefixBlock, 0, s>>>(H, S.n_pchunks, visits);
    DT_HIP(hipGetLastError());
    k_heavy_prefix_scan<<<dim3(grid_for(npc, 256), k), 256, 0, s>>>(H, S.n_pchunks);
    DT_HIP(hipGetLastError());
    k_heavy_prefix_add<<<dim3(pgrid, k), kPrefixBlock, 0, s>>>(H, S.n_pchunks);
    prof_end(ctx, kProfHeavyPrefix, s);
    DT_HIP(hipGetLastError());
    prof_begin(ctx, kProfHeavyCount, s);
    k_heavy_count<ACC, 256><<<dim3(hg, k), 256, 0, s>>>(H, hr.cb, S.n_chunks, part, cells_dev, visits);
    prof_end(ctx, kProfHeavyCount, s);
    DT_HIP(hipGetLastError());
    return DT_OK;
}

// The four paths' kernels of a planned count with accumulator ACC: the heavy ones on sl, and the light
// ones before them on sl, the medium one on sm and the unit one on s, or, with `small`, these three in one
// launch on s; partial slots of 8 words (16 for AccW): heavy, then medium, light, unit.
template <class ACC>
int launch_paths(dt_graph *g, const DQuery &q, const CountPlan &p, const ScratchView &sv, bool small, hipStream_t s,
                 hipStream_t sl, hipStream_t sm, int64_t *cells_dev, unsigned long long *visits) {
    dt_ctx *ctx = g->ctx;
    Schedule &S = g->sched;
    constexpr uint64_t W = std::is_same<ACC, AccW>::value ? 16 : 8;
    const unsigned lg = p.lg, hg = p.hg, mg = p.mg, ug = p.ug;
    int64_t *hp = sv.part, *mp = hp + W * hg, *lp = mp + W * mg, *up = lp + W * lg;
    const uint32_t *eoff = g->eoff.as<uint32_t>();
    const uint64_t *key = g->key.as<uint64_t>();
    if constexpr (!kCellsAcc<ACC>) {
        if (small) {
            SmallCount C{p.lr, p.mr, p.light, p.medium, p.mitems, eoff, p.mlev, key, S.unit.as<uint4>(), p.ub, p.ue, q,
                         unit_query(q), mg, lg, ug};
            k_small<ACC, 256><<<mg + lg + ug, 256, 0, s>>>(C, mp);
            DT_HIP(hipGetLastError());
            if (p.hr.n) DT_TRY(launch_heavy<ACC>(g, &q, 1, p.hr, hg, sv.heavy, hp, sl, nullptr, nullptr));
            return DT_OK;
        }
    }
    if (lg) {
        prof_begin(ctx, kProfLight, sl);
        k_light<ACC, kLightBlock><<<lg, kLightBlock, 0, sl>>>(p.lr, p.light, eoff, key, q, lp, cells_dev, visits);
        prof_end(ctx, kProfLight, sl);
        DT_HIP(hipGetLastError());
    }
    if (mg) {
        prof_begin(ctx, kProfMedium, sm);
        // shared where a triangle's close pairs are a fair part of all its pairs: deltas from 1/128 of the
        // span on (61M edges: 1/240 of it 545 us with either, 1/2800 418 shared and 410 not, none 1700 and
        // 2400); not for 128-bit sums, whose LDS would leave one block a compute unit
        bool shared = false;
        if constexpr (std::is_same<ACC, Acc<false>>::value) shared = q.d13 >= g->span / 128;
        if (shared)
            k_medium_shared<512><<<std::min(mg, grid_for(p.mr.pre[p.mr.n], 512)), 512, 0, sm>>>(
                p.mr, p.medium, p.mitems, p.mlev, eoff, key, q, mp, mg, visits);
        else
            k_medium<ACC, 256><<<mg, 256, 0, sm>>>(p.mr, p.medium, p.mitems, p.mlev, eoff, key, q, mp, cells_dev, visits);
        prof_end(ctx, kProfMedium, sm);
        DT_HIP(hipGetLastError());
    }
    if (ug) {
        const UQuery u = unit_query(q);
        prof_begin(ctx, kProfUnit, s);
        k_unit<ACC, kUnitBlock><<<ug, kUnitBlock, 0, s>>>(p.ub, p.ue, S.unit.as<uint4>(), u, up, cells_dev, visits);
        prof_end(ctx, kProfUnit, s);
        DT_HIP(hipGetLastError());
    }
    if (p.hr.n) DT_TRY(launch_heavy<ACC>(g, &q, 1, p.hr, hg, sv.heavy, hp, sl, cells_dev, visits));
    return DT_OK;
}

// Enqueue one planned count on stream s: partials -> out8_dev (int64[8]); cells mode accumulates the
// 48 cells into cells_dev (zeroed here) instead.  The scratch must hold the plan's needs.  With
// visits, the kernels add the pairs and list elements they iterate over to *visits.
int count_launch(dt_graph *g, const DQuery &q, const CountPlan &p, int64_t *out8_dev, hipStream_t s, bool cells,
                 int64_t *cells_dev, const ScratchView &sv, unsigned long long *visits) {
    dt_ctx *ctx = g->ctx;
    prof_clear(ctx, false);
    if (sv.part_bytes < p.part_bytes || sv.heavy_bytes < p.heavy_bytes)
        return fail(DT_EINVAL, "count scratch too small (%zu of %zu, %zu of %zu bytes)", sv.part_bytes, p.part_bytes,
                    sv.heavy_bytes, p.heavy_bytes);
    const unsigned lg = p.lg, hg = p.hg, mg = p.mg, ug = p.ug;
    const uint64_t n_part = p.n_part;
    int64_t *part = sv.part;
    if (cells) {
        k_zero<<<1, 64, 0, s>>>(48, cells_dev);
        DT_HIP(hipGetLastError());
    }
    // The paths are independent (each writes its own partial slots): when more than one has work,
    // the light and then the heavy kernels run on the context's first side stream and the medium
    // kernel on the second, forked from s here and joined back before the reduction, beside the
    // unit kernel on s, so that their latency-bound tails overlap.  A small count takes the light,
    // medium and unit blocks in one launch on s, and only the heavy kernels beside it (not while it is
    // profiled, so that each path has its time).
    const bool small = !cells && !visits && !ctx->prof && (lg || mg || ug) &&
                       (uint64_t)lg + mg + ug <= (uint64_t)ctx->num_cus * kSmallPerCu;
    hipStream_t sl = s, sm = s;
    const bool fork = ctx->side[0] && (small ? hg != 0 : ((lg || hg ? 1 : 0) + (mg ? 1 : 0) + (ug ? 1 : 0)) >= 2);
    const bool fork_l = fork && (hg || (!small && lg)), fork_m = fork && !small && mg;
    if (fork) {
        DT_HIP(hipEventRecord(ctx->ev_fork, s));
        if (fork_l) {
            DT_HIP(hipStreamWaitEvent(ctx->side[0], ctx->ev_fork, 0));
            sl = ctx->side[0];
        }
        if (fork_m) {
            DT_HIP(hipStreamWaitEvent(ctx->side[1], ctx->ev_fork, 0));
            sm = ctx->side[1];
        }
    }
    if (cells) {
        DT_TRY(launch_paths<Acc<true>>(g, q, p, sv, small, s, sl, sm, cells_dev, visits));
    } else if (p.wide) {
        DT_TRY(launch_paths<AccW>(g, q, p, sv, small, s, sl, sm, nullptr, visits));
    } else {
        DT_TRY(launch_paths<Acc<false>>(g, q, p, sv, small, s, sl, sm, nullptr, visits));
    }
    if (fork_l) {
        DT_HIP(hipEventRecord(ctx->ev_join[0], sl));
        DT_HIP(hipStreamWaitEvent(s, ctx->ev_join[0], 0));
    }
    if (fork_m) {
        DT_HIP(hipEventRecord(ctx->ev_join[1], sm));
        DT_HIP(hipStreamWaitEvent(s, ctx->ev_join[1], 0));
    }
    if (!cells) {
        prof_begin(ctx, kProfReduce, s);
        if (p.wide) k_reduce_w<<<1, 256, 0, s>>>(n_part, part, out8_dev);
        else k_reduce<<<1, kReduceBlock, 0, s>>>(n_part, part, out8_dev);
        prof_end(ctx, kProfReduce, s);
        DT_HIP(hipGetLastError());
    }
    return DT_OK;
}

// Plan one count, grow the scratch sc to its needs, and enqueue it on stream s.
int count_enqueue(dt_graph *g, const DQuery &q, int64_t *out8_dev, hipStream_t s, bool cells,
                  int64_t *cells_dev, Scratch &sc, unsigned parts, unsigned long long *visits) {
    CountPlan p;
    count_plan(g, q, parts, p);
    DT_TRY(ensure(g->ctx, sc.partials, p.part_bytes));
    if (p.heavy_bytes) DT_TRY(ensure(g->ctx, sc.heavy_vals, p.heavy_bytes));
    ScratchView sv;
    sv.part = sc.partials.as<int64_t>();
    sv.part_bytes = sc.partials.bytes;
    sv.heavy = sc.heavy_vals.as<uint8_t>();
    sv.heavy_bytes = p.heavy_bytes ? sc.heavy_vals.bytes : 0;
    return count_launch(g, q, p, out8_dev, s, cells, cells_dev, sv, visits);
}

void count_reduce(uint64_t n_part, const int64_t *part, int64_t *out8_dev, hipStream_t s) {
    k_reduce<<<1, kReduceBlock, 0, s>>>(n_part, part, out8_dev);
}

// A sweep: k <= kSweepMax queries with one window.  The unit, light and medium kernels visit each
// triangle's data once per pass and count it for every delta triple: records and lists are read
// once, the light path enumerates each triangle's pairs once, the medium path finds each entry's
// close pairs once (for the largest d13); only the delta-dependent searches repeat.  The rare heavy
// triangles are counted for every query in one set of launches (61M edges, eight triples: 1.3 ms of 1.9
// when each query took its own, one after the other).
int count_sweep_enqueue(dt_graph *g, const DQuery *qs, uint32_t k, int64_t *out_dev, hipStream_t s, Scratch &sc,
                        DevMem &heavy) {
    dt_ctx *ctx = g->ctx;
    Schedule &S = g->sched;
    if (k == 0 || k > kSweepMax) return fail(DT_EINVAL, "a sweep pass takes 1..%u queries", kSweepMax);
    SweepQ Q{};
    Q.k = k;
    Q.d13max = 0;
    for (uint32_t j = 0; j < k; ++j) {
        Q.q[j] = qs[j];
        Q.u[j] = unit_query(qs[j]);
        Q.d13max = qs[j].d13 > Q.d13max ? qs[j].d13 : Q.d13max;
    }
    const DQuery &q0 = qs[0];   // the window (and so every range) is the same for all k
    // one medium / heavy split for the whole pass: the level of the largest d13 (the medium pass
    // finds close pairs at that distance for every triple)
    uint32_t qlm = 0;
    for (uint32_t j = 0; j < k; ++j) qlm = qs[j].qlev > qlm ? qs[j].qlev : qlm;
    DQuery qh = q0;
    qh.qlev = qlm;
    HeavyRange hr;
    heavy_range(g, qh, hr);
    const unsigned hg = hr.n ? (unsigned)std::min<uint64_t>(S.n_chunks - hr.cb, (uint64_t)ctx->num_cus * 16) : 0;
    Q.qlev = qlm;
    Ranges lr, mr;
    const uint8_t *mlev = nullptr;
    cell_ranges(S.light_cells, S.cell_shift, q0, lr);
    medium_ranges(g, qh, mr, &mlev);
    const uint64_t nl = lr.pre[lr.n], nmi = mr.pre[mr.n];
    const uint32_t *light = (q0.windowed ? S.light_w : S.light).as<uint32_t>();
    const uint32_t *medium = (q0.windowed ? S.medium_w : S.medium).as<uint32_t>();
    const uint32_t *mitems = (q0.windowed ? S.mitems_w : S.mitems).as<uint32_t>();
    const unsigned lg = nl ? (unsigned)std::min<uint64_t>((nl + kLightBlock - 1) / kLightBlock, (uint64_t)ctx->num_cus * 16) : 0;
    const unsigned lgx = lg ? ((lg + 7) / 8) * 8 : 0;
    const unsigned mg = nmi ? (unsigned)std::min<uint64_t>((nmi + 255) / 256, (uint64_t)ctx->num_cus * 8) : 0;
    uint64_t ub = 0, ue = 0;
    if (S.n_unit) unit_range(g, q0, &ub, &ue);
    const unsigned ug = ue > ub ? (unsigned)std::min<uint64_t>((ue - ub + kUnitPerBlock - 1) / kUnitPerBlock,
                                                               (uint64_t)ctx->num_cus * 8) : 0;
    const uint64_t n_slot = (uint64_t)ug + lgx + mg;
    DT_TRY(ensure(ctx, sc.sweep_partials, (n_slot + hg + 1) * k * 8 * sizeof(int64_t)));
    int64_t *part = sc.sweep_partials.as<int64_t>(), *hpart = part + 8 * n_slot * k;
    // the heavy triangles of all k queries in one set of launches, when their scratch may be had: a
    // query's prefix arrays each, at most kSweepHeavyBytes (and half a budget) of them at a time, else one
    // query after the other
    uint32_t hk = 0;
    uint8_t *hscratch = nullptr;
    if (hg) {
        const uint64_t most = ctx->budget ? std::min<uint64_t>(kSweepHeavyBytes, ctx->budget / 2) : kSweepHeavyBytes;
        hk = (uint32_t)std::min<uint64_t>(k, std::max<uint64_t>(1, most / hr.scratch_bytes));
        const size_t bytes = hk * hr.scratch_bytes;
        if (hk > 1 && heavy.bytes < bytes) {
            heavy.reset();
            const int rc = pool_room(ctx, bytes) ? dev_alloc(ctx, heavy, bytes) : DT_ENOMEM;
            if (rc != DT_OK && rc != DT_ENOMEM) return rc;
            if (rc == DT_ENOMEM) {
                clear_error();
                hk = 1;
            }
        }
        if (hk == 1) DT_TRY(ensure(ctx, sc.heavy_vals, hr.scratch_bytes));
        hscratch = (hk > 1 ? heavy : sc.heavy_vals).as<uint8_t>();
    }
    // the light (then heavy) and medium passes run on the side streams, beside the unit pass (as in a
    // count)
    hipStream_t sl = s, sm = s;
    const bool fork = ctx->side[0] && ((ug ? 1 : 0) + (lgx || hg ? 1 : 0) + (mg ? 1 : 0)) >= 2;
    if (fork) {
        DT_HIP(hipEventRecord(ctx->ev_fork, s));
        if (lgx || hg) {
            DT_HIP(hipStreamWaitEvent(ctx->side[0], ctx->ev_fork, 0));
            sl = ctx->side[0];
        }
        if (mg) {
            DT_HIP(hipStreamWaitEvent(ctx->side[1], ctx->ev_fork, 0));
            sm = ctx->side[1];
        }
    }
    if (ug) {
        prof_begin(ctx, kProfUnit, s);
        k_unit_sweep<kUnitBlock><<<ug, kUnitBlock, 0, s>>>(ub, ue, S.unit.as<uint4>(), Q, part, 0);
        prof_end(ctx, kProfUnit, s);
        DT_HIP(hipGetLastError());
    }
    if (lgx) {
        prof_begin(ctx, kProfLight, sl);
        k_light_sweep<kLightBlock><<<lgx, kLightBlock, 0, sl>>>(lr, light, g->eoff.as<uint32_t>(), g->key.as<uint64_t>(),
                                                                Q, part, ug);
        prof_end(ctx, kProfLight, sl);
        DT_HIP(hipGetLastError());
    }
    for (uint32_t j = 0; hg && j < k; j += hk) {
        const uint32_t kk = std::min(hk, k - j);
        DT_TRY(launch_heavy<Acc<false>>(g, qs + j, kk, hr, hg, hscratch, hpart + 8ull * hg * j, sl,
                                        nullptr, nullptr));
    }
    if (mg) {
        prof_begin(ctx, kProfMedium, sm);
        k_medium_sweep<256><<<mg, 256, 0, sm>>>(mr, medium, mitems, mlev, g->eoff.as<uint32_t>(), g->key.as<uint64_t>(),
                                                Q, part, (uint64_t)ug + lgx);
        prof_end(ctx, kProfMedium, sm);
        DT_HIP(hipGetLastError());
    }
    if (fork) {
        if (lgx || hg) {
            DT_HIP(hipEventRecord(ctx->ev_join[0], sl));
            DT_HIP(hipStreamWaitEvent(s, ctx->ev_join[0], 0));
        }
        if (mg) {
            DT_HIP(hipEventRecord(ctx->ev_join[1], sm));
            DT_HIP(hipStreamWaitEvent(s, ctx->ev_join[1], 0));
        }
    }
    prof_begin(ctx, kProfReduce, s);
    k_reduce_sweep<<<k, kReduceBlock, 0, s>>>(n_slot, k, part, hg, hpart, out_dev);
    prof_end(ctx, kProfReduce, s);
    DT_HIP(hipGetLastError());
    return DT_OK;
}

}  // namespace dt
