// Degeneracy ordering by a parallel k-core peel (Section 3, the degeneracy ordering: vertices taken
// in order of smallest remaining degree; the degeneracy is the largest core number).
//
// Level k removes every remaining vertex whose remaining degree is <= k: the vertices found by a
// scan of the remaining ones, then those whose degree falls to k while their neighbours are
// removed.  A vertex takes its position in the ordering no later than the start of its own
// removal, and positions are handed out in time order.  When v is queued at most k of its
// neighbours are not yet removed; a neighbour placed after v started its removal after v was
// placed, hence after v was queued, so it is one of those: the out-degree of v in G_prec is at
// most k = core(v) <= degeneracy, the property Theorem 1's bound rests on.  (Different removal
// orders give different orientations but the same counts: each static triangle is counted once
// under its own naming u < v < w.)
//
// The whole peel is one cooperative (co-resident) grid: levels and rounds are separated by grid
// barriers instead of kernel launches and host round trips, since power-law graphs need thousands
// of removal steps, most with frontiers of a few vertices.  Within a level, a block removes the
// vertices its own removals queued right away (a cascade local to the block, with workgroup
// barriers only), so a grid round usually ends a level; only vertices queued past a full staging
// list wait for another round.  The first levels remove most of the graph and are bound by work,
// the later ones by latency, and a barrier's cost grows with the number of blocks that meet at it:
// the grid starts with one block of 1024 threads per CU and narrows to 128, then 64 blocks as vertices
// run out and levels grow small, and hands its last 65,536 vertices to a finish that takes no levels
// (below), or back to the levels where that is the slower way.  The barrier counts arrivals in groups of
// blocks.  Counters that decide the next step (queue positions taken in a phase, survivors of a level scan)
// rotate over three slots, so a fast block starting the next phase never changes what a slow block reads,
// and every block takes the same branch.  A vertex is queued at most
// once: by the level scan when its degree is <= k (no decrement runs during a scan), or by the
// single decrement that takes its degree from k + 1 to k (degrees only fall, and a queued vertex
// already has degree <= k, so no later decrement can see k + 1 again); a vertex queued by a
// decrement also gets a large negative degree, so that the next scans, which still list it, skip
// it.  The queue index is also bounds-checked, the host checks that exactly n vertices were queued, and
// the pass that takes the ranks from the queue that every place of it was taken.  A barrier that waits
// far longer than any peel could take sets an error flag and lets its block go, so that a fault in this
// logic ends the kernel instead of hanging it.
#include <algorithm>
#include <type_traits>

#include "finish_room.h"
#include "internal.h"

namespace dt {

namespace {

constexpr unsigned kBlock = 1024;
constexpr unsigned kGridWide = 256;    // blocks of the first levels
// The grid narrows as vertices run out (blocks while at least `from` remain), where a level removes fewer
// than kBusy of them: its rounds then wait for each other more than they work, and fewer blocks meet
// sooner (61M edges, whose levels grow small: 3.9 ms so, 4.3 with 256 blocks throughout; 10M edges, a few
// large levels: 0.50 ms so, 0.61 narrowing by the vertices left alone).
struct Width {
    uint32_t from;
    unsigned blocks;
};
constexpr Width kWidths[3] = {{400000, kGridWide}, {50000, 128}, {0, 64}};
constexpr uint32_t kBusy = 32768;
// LDS words of a peel block: two staging halves, the vertices the block is removing and those their
// removal queues
constexpr uint32_t kLdsWords = 40800;
constexpr uint32_t kStage = kLdsWords / 2;
constexpr uint32_t kUnset = 0xffffffffu;
constexpr long kSpinLimit = 1l << 26;
// degree of a vertex queued during removal rounds: negative, and it stays negative under the
// at most n further decrements, so a level scan never takes it again
constexpr int kRemoved = -(1 << 30);

struct PeelCtl {
    unsigned int qtail;      // vertices queued in all (written at the end)
    unsigned int qc[3];      // per grid phase mod 3: queue positions taken in that phase
    unsigned int ovc[3];     // per grid phase mod 3: vertices that phase queued past a full stage
    unsigned int error;      // a barrier gave up waiting, or a consistency check failed
    unsigned int rounds;     // removal rounds
    unsigned int kappa;      // largest level that removed a vertex
    unsigned int fin[3];     // finish, per phase mod 3: a bound fell
    unsigned int left;       // the finish left its vertices to the level peel
    unsigned long long lres; // hand-over: local ids (low word) and adjacency entries (high word) given out
    unsigned int ho;         // 1: the grid handed its last vertices over (the state below is set)
    unsigned int ho_tail, ho_k, ho_rounds;   // queue positions taken, level and rounds at the hand-over
    unsigned int scan[3][2]; // per level mod 3: survivors of the level scan, their smallest degree
};

__device__ __forceinline__ unsigned ld_relaxed(const unsigned *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_relaxed(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Grid barrier.  Arrivals are counted per group of kBarGroup blocks, the last of a group arrives at the
// root, and every block polls the root, or the only group's counter: an atomic on one address takes
// about 15 ns, so 256 arrivals at one counter, which the pollers read meanwhile, took 4 us and more
// (the level peel of 61M edges with one counter 5.0 ms, 3.9 so).
// Counters only ever increase, and every block passes the same barriers in the same order with the same
// participants (the grid narrows by whole groups), so a barrier is complete once its counter holds the
// running sum of its arrivals: a block's first thread publishes its block's writes, arrives, polls (an
// acquiring poll would throw away its caches each time) and takes the others' writes; no block has to
// release the others.  A barrier that waits far longer than any peel could take sets an error flag and
// lets its block go.
constexpr unsigned kBarGroup = 32;   // blocks that share a counter
constexpr unsigned kBarLine = 32;    // words between counters
constexpr unsigned kBarWords = (1 + 1024 / kBarGroup) * kBarLine;   // the root, then one per group
struct BarTurn {
    unsigned turn = 0, root = 0;   // barriers passed, arrivals at the root so far
};
__device__ void group_barrier(unsigned *bar, unsigned *error, unsigned nblk, BarTurn &b) {
    const unsigned groups = (nblk + kBarGroup - 1) / kBarGroup;
    ++b.turn;
    b.root += groups > 1 ? groups : 0u;
    __syncthreads();
    if (threadIdx.x == 0 && nblk > 1) {
        __threadfence();
        const unsigned grp = blockIdx.x / kBarGroup;
        const unsigned size = grp + 1 < groups ? kBarGroup : nblk - grp * kBarGroup;
        unsigned *mine = &bar[(1 + grp) * kBarLine];
        unsigned *poll = groups > 1 ? &bar[0] : mine;
        const unsigned target = groups > 1 ? b.root : b.turn * size;
        if (atomicAdd(mine, 1u) + 1 == b.turn * size && groups > 1) {
            __threadfence();
            atomicAdd(&bar[0], 1u);
        }
        long spins = 0;
        while (ld_relaxed(poll) < target) {
            __builtin_amdgcn_s_sleep(1);
            ++spins;
            // (a block that found an error has left)
            if ((spins & 1023) == 0 && ld_relaxed(error)) break;
            if (spins > kSpinLimit) {
                atomicOr(error, 1u);
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

// A vertex whose degree a removal took from k + 1 to k joins the block's staging list, which the
// same block removes next (its position in the ordering is taken then); a full staging list sends
// the rest to the overflow list, which the next grid phase takes.
__device__ __forceinline__ void enqueue(uint32_t v, uint32_t k, uint32_t n, uint32_t *level, int *deg,
                                        unsigned *ovc, uint32_t *ovf, unsigned *err, uint32_t *s_stage,
                                        unsigned *s_cnt) {
    level[v] = k;
    __hip_atomic_store(&deg[v], kRemoved, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t p = atomicAdd(s_cnt, 1u);
    if (p < kStage) {
        s_stage[p] = v;
    } else {
        const uint32_t o = atomicAdd(ovc, 1u);
        if (o < n) ovf[o] = v;
        else atomicOr(err, 8u);
    }
}

__device__ __forceinline__ unsigned wave_min(unsigned x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned y = __shfl_xor(x, o, 64);
        x = y < x ? y : x;
    }
    return x;
}

// remove the adjacency entries [b, e) of one vertex (this lane: first, first + stride, ...)
__device__ __forceinline__ void remove_range(uint32_t b, uint32_t e, uint32_t first, uint32_t stride, uint32_t k,
                                             uint32_t n, const uint32_t *__restrict__ col, int *__restrict__ deg,
                                             uint32_t *__restrict__ level, unsigned *ovc, uint32_t *ovf,
                                             unsigned *err, uint32_t *s_stage, unsigned *s_cnt) {
    uint32_t j = b + first;
    // four independent decrements in flight per lane
    for (; j + 3 * stride < e; j += 4 * stride) {
        const uint32_t x0 = col[j], x1 = col[j + stride], x2 = col[j + 2 * stride], x3 = col[j + 3 * stride];
        const int o0 = atomicSub(&deg[x0], 1), o1 = atomicSub(&deg[x1], 1), o2 = atomicSub(&deg[x2], 1),
                  o3 = atomicSub(&deg[x3], 1);
        if (o0 == (int)k + 1) enqueue(x0, k, n, level, deg, ovc, ovf, err, s_stage, s_cnt);
        if (o1 == (int)k + 1) enqueue(x1, k, n, level, deg, ovc, ovf, err, s_stage, s_cnt);
        if (o2 == (int)k + 1) enqueue(x2, k, n, level, deg, ovc, ovf, err, s_stage, s_cnt);
        if (o3 == (int)k + 1) enqueue(x3, k, n, level, deg, ovc, ovf, err, s_stage, s_cnt);
    }
    for (; j < e; j += stride) {
        const uint32_t x = col[j];
        const int old = atomicSub(&deg[x], 1);
        if (old == (int)k + 1) enqueue(x, k, n, level, deg, ovc, ovf, err, s_stage, s_cnt);
    }
}

__device__ __forceinline__ void remove_edges(uint32_t v, uint32_t first, uint32_t stride, uint32_t k,
                                             uint32_t n, const uint32_t *__restrict__ row,
                                             const uint32_t *__restrict__ col, int *__restrict__ deg,
                                             uint32_t *__restrict__ level, unsigned *ovc, uint32_t *ovf,
                                             unsigned *err, uint32_t *s_stage, unsigned *s_cnt) {
    remove_range(row[v], row[v + 1], first, stride, k, n, col, deg, level, ovc, ovf, err, s_stage, s_cnt);
}

// ------------------------------------------------------------------------------------------------
// The finish: the last R vertices, on the subgraph they induce (local 16-bit ids; rows lrow, lcol).
//
// Level after level would take hundreds of levels of a few removal rounds each, bound by the latency
// of every round.  Their core numbers come instead from bounds that fall: every vertex holds an upper
// bound of its core number, first its degree, and replaces it by the largest t such that t neighbours
// have bounds of at least t, until no bound falls (the last bounds are the core numbers).  A phase reads
// the bounds that the phase before left, so the phase in which a bound takes its last value orders its
// shell: when v's bound fell to core(v), at most core(v) of its neighbours had larger ones, and those of
// v's shell that fell to their core numbers in the same phase or later, like all of larger cores, were
// among them.  Vertices ordered by (core, phase) are therefore in degeneracy order, and no vertex need be
// removed from the others' counts.  Those of one shell and phase come by classes of their degree over the
// core number, hubs last, as the levels would remove them: a hub before its shell's other vertices is the
// source of all their triangles, with its long edge lists (40,000 vertices of a power law whose hubs share
// pairs: prefix arrays of 2.3M to 3.7M slots in any order, 1.6M to 2.0M so, 1.8M by levels).
//
// 57 to 77 phases for the last 65,536 vertices of 61M-edge graphs, where levels took 410 and 2,000 rounds
// (one's peel then 13.9 ms, now 6.7, 2.3 of them here; 2.8 with a second part of 50 phases that removed the
// shells' vertices in rounds, at 1.3M edges 0.36 against 0.26 ms).  A finish whose falls do not die down
// leaves its vertices to the levels (kSlowPhase below).  65,536 is what 16-bit ids and one workgroup's LDS
// hold; above it the level peel is the faster one (a level of many vertices there costs less than their
// share of those phases).
//
// A wavefront owns consecutive local ids holding an even share of the entries.  Every phase each block
// copies all bounds (128 KB at most) into LDS, where the gathers along the rows go; rows stream from
// L2, short rows packed 64 entries at a time, rows of up to kRegRow entries held in registers
// while their new bound is searched by ballots.  Bounds have two buffers, one read and one written.
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kGroup = 32;      // vertices of a wavefront handled at once
constexpr uint32_t kVertexCost = 32; // a vertex's share of the work, in entries, besides its row
constexpr uint32_t kPerWave = 16;    // vertices per wavefront that a grid is sized for
constexpr uint32_t kPiece = 128;     // entries of a row a wavefront reads at once, two a lane
constexpr uint32_t kRegPieces = 8;   // pieces of a row held in registers
constexpr uint32_t kRegRow = kPiece * kRegPieces;
constexpr uint32_t kFinSmall = 1024; // up to this many vertices one block finishes alone
// When the finish leaves its vertices to the levels: after phase kSlowPhase if more than a quarter as many
// bounds still fall as in the first; when kFewPhases phases, seen every kTellPhases, had at most kFewFell
// falls each and none more than twice those of the first; and after kPhaseMost phases.  Where degrees are
// spread, falls are a fifteenth of the first ones by phase 8 (61M edges; random graphs, preferential
// attachment, small worlds, points in a plane: 1/9 to 1/1700), then few and growing until they burst again
// and again (seven 61M-edge graphs: such rows of at most 16 phases, small worlds 21), and the phases at most
// 77.  On a chain or a lattice they go on as they began (a path of 60,000 vertices: 2 a phase for 30,000
// phases, 373 ms by them all, 42 ms left to the levels; a 1,000-vertex path beside a 40,000-vertex power law:
// 15.4 and 4.5 ms; a lattice of 250 x 250: 4.2 and 1.9), so that the phases tried cost little beside the
// levels.
constexpr uint32_t kTellPhases = 8, kSlowPhase = 8, kFewFell = 64, kFewPhases = 48, kPhaseMost = 192;
static_assert(kSlowPhase % kTellPhases == 0 && kFewPhases % kTellPhases == 0, "falls are told then");
constexpr uint32_t kSharedRows = 16; // rows at most that a block's wavefronts walk together
constexpr uint32_t kSlots = 2048;    // places a block takes together

struct FinArgs {
    const uint32_t *rlist, *lrow;
    const uint16_t *lcol;
    uint16_t *val;        // two buffers of R bounds
    uint32_t *base;       // first position of each cell: core, phase and class of degree
    uint32_t *cur;        // positions taken in each
    uint32_t *when;       // the last phase in which each vertex's bound fell, and one (0: in none), then its cell
    uint32_t *pos;        // position of each vertex among those of its cell
    uint32_t *level, *queue;
    uint32_t *falls;      // bounds that fell in a phase, by block: two buffers
    unsigned *bar;        // barrier counters (kBarWords)
    PeelCtl *ctl;
};

// Barrier of the finish's nblk blocks; the error state comes back in *s_err, read once every block has
// arrived.
__device__ void fin_barrier(const FinArgs &A, unsigned nblk, BarTurn &turn, unsigned *s_err) {
    group_barrier(A.bar, &A.ctl->error, nblk, turn);
    if (threadIdx.x == 0) *s_err = ld_relaxed(&A.ctl->error);
    __syncthreads();
}

// f(I) for every piece I that begins before entry d: nested, so that one jump skips the rest
template <uint32_t I = 0, class F> __device__ __forceinline__ void pieces(uint32_t d, F f) {
    if constexpr (I < kRegPieces) {
        if (I * kPiece < d) {
            f(std::integral_constant<uint32_t, I>());
            pieces<I + 1>(d, f);
        }
    }
}
// The first kRegRow of d entries at b, two a lane and piece (the last piece may read past the end, into
// the next row or the list's padding), and their values in s_v: 0 past the end, below every threshold
// asked of them.
__device__ __forceinline__ void row_entries(const uint16_t *__restrict__ lcol, uint32_t b, uint32_t d, unsigned lane,
                                            uint32_t (&c)[kRegPieces]) {
    pieces(d, [&](auto i) { __builtin_memcpy(&c[i], lcol + b + i * kPiece + 2 * lane, 4); });
}
__device__ __forceinline__ void row_values(const uint16_t *s_v, const uint32_t (&c)[kRegPieces], uint32_t d, unsigned lane,
                                           uint32_t (&v)[2 * kRegPieces]) {
    pieces(d, [&](auto i) {
        const uint32_t j = i * kPiece + 2 * lane;
        const uint32_t x = s_v[c[i] & 0xffffu], y = s_v[c[i] >> 16];
        v[2 * i] = j < d ? x : 0u;
        v[2 * i + 1] = j + 1 < d ? y : 0u;
    });
}
// values of at least t >= 1 among them
__device__ __forceinline__ uint32_t count_at_least(const uint32_t (&v)[2 * kRegPieces], uint32_t d, uint32_t t) {
    uint32_t n = 0;
    pieces(d, [&](auto i) {
        n += (uint32_t)__popcll(__ballot(v[2 * i] >= t)) + (uint32_t)__popcll(__ballot(v[2 * i + 1] >= t));
    });
    return n;
}
// f(values, entries left) for the first kRegRow entries of a row (in c), then the next ones, while f
// says to go on; the entries of the next stretch are read while f works on one
template <class F>
__device__ __forceinline__ void row_stretches(const uint16_t *__restrict__ lcol, const uint16_t *s_v, uint32_t b, uint32_t d,
                                              unsigned lane, const uint32_t (&first)[kRegPieces], F f) {
    uint32_t c[kRegPieces];
#pragma unroll
    for (uint32_t i = 0; i < kRegPieces; ++i) c[i] = first[i];
    for (uint32_t j0 = 0;; j0 += kRegRow) {
        const uint32_t left = d - j0;
        uint32_t nx[kRegPieces], v[2 * kRegPieces];
        if (left > kRegRow) row_entries(lcol, b + j0 + kRegRow, left - kRegRow, lane, nx);
        row_values(s_v, c, left, lane, v);
        if (!f(v, left) || left <= kRegRow) return;
#pragma unroll
        for (uint32_t i = 0; i < kRegPieces; ++i) c[i] = nx[i];
    }
}

// The rows of up to kGroup consecutive vertices.
struct GroupRows {
    uint32_t rows;      // lane l <= nv: first entry of vertex l (the end of the last at l = nv)
    uint32_t nv;
    __device__ __forceinline__ uint32_t begin(uint32_t x) const { return __builtin_amdgcn_readlane(rows, x); }
    // lane l: end of the l-th row from x on, relative to the first (far past 64 beyond the group)
    __device__ __forceinline__ uint32_t ends(uint32_t x, uint32_t b, unsigned lane) const {
        const uint32_t e = __shfl(rows, (x + 1 + lane) & 63, 64);
        return x + 1 + lane <= nv ? e - b : 0x7fffffffu;
    }
};

// lane's row among the packed ones (ends per lane, cnt of them): how many end at or before it
__device__ __forceinline__ uint32_t pack_row(uint32_t ends, uint32_t cnt, unsigned lane) {
    uint32_t r = 0;
#pragma unroll
    for (uint32_t s = kGroup; s > 0; s >>= 1) {
        const uint32_t e = __shfl(ends, (r + s - 1) & 63, 64);
        if (r + s <= cnt && e <= lane) r += s;
    }
    return r;
}

__device__ __forceinline__ uint64_t bits_between(uint32_t a, uint32_t b) {   // bits [a, b), b <= 64
    return (b < 64 ? (1ull << b) - 1 : ~0ull) & ~(a < 64 ? (1ull << a) - 1 : ~0ull);
}

// Walks the rows of a group: rows that fit 64 entries together by pack(x, cnt, b, ends), a longer one
// by row(x, b, d, c) with its first entries in c; the entries of a long row are read while the one
// before it is worked on.
template <class Pack, class Row>
__device__ __forceinline__ void walk_rows(const GroupRows &G, const uint16_t *__restrict__ lcol, unsigned lane, Pack pack,
                                          Row row) {
    uint32_t c[kRegPieces], x = 0;
    bool have = false;
    while (x < G.nv) {
        const uint32_t b = G.begin(x), ends = G.ends(x, b, lane);
        const uint64_t fits = __ballot(ends <= 64);
        const uint32_t cnt = (uint32_t)__ffsll((unsigned long long)~fits) - 1;   // (lane 63 never fits)
        if (cnt > 0) {
            pack(x, cnt, b, ends);
            x += cnt;
            have = false;
            continue;
        }
        const uint32_t d = __builtin_amdgcn_readlane(ends, 0);
        if (!have) row_entries(lcol, b, d, lane, c);
        uint32_t nx[kRegPieces];
        have = x + 1 < G.nv;
        if (have) {
            const uint32_t nb = G.begin(x + 1), nd = G.begin(x + 2) - nb;
            have = nd > 64;
            if (have) row_entries(lcol, nb, nd, lane, nx);
        }
        row(x, b, d, c);
#pragma unroll
        for (uint32_t i = 0; i < kRegPieces; ++i) c[i] = nx[i];
        x += 1;
    }
}

// New bounds of a group's vertices (lane x < nv: vertex x; its present bound h comes in), at least k0.
// Rows of `shared` entries and more keep theirs (the block walks those together).
__device__ __forceinline__ uint32_t group_bounds(const GroupRows &G, const uint16_t *__restrict__ lcol,
                                                 const uint16_t *s_h, uint32_t h, uint32_t k0, uint32_t shared,
                                                 unsigned lane) {
    walk_rows(
        G, lcol, lane,
        [&](uint32_t x, uint32_t cnt, uint32_t b, uint32_t ends) {
            const uint32_t len = __builtin_amdgcn_readlane(ends, cnt - 1);
            const uint32_t r = pack_row(ends, cnt, lane);
            const uint32_t H = __shfl(h, (x + r) & 63, 64);
            const uint32_t prev = __shfl(ends, (r - 1) & 63, 64), end = __shfl(ends, r & 63, 64);
            const uint32_t beg = r ? prev : 0u;
            const bool in = lane < len;
            const uint32_t v = in ? s_h[lcol[b + lane]] : 0u;
            const uint64_t mine = in ? bits_between(beg, end) : 0ull;
            const uint32_t c = (uint32_t)__popcll(__ballot(in && v >= H) & mine);
            uint32_t lo = H, hi = H;
            if (in && c < H) {
                lo = c > k0 ? c : k0;
                hi = H - 1;
                if (lo > hi) lo = hi;   // (a bound is never below k0)
            }
            while (__ballot(lo < hi)) {
                const uint32_t mid = (lo + hi + 1) >> 1;
                const uint32_t cm = (uint32_t)__popcll(__ballot(in && v >= mid) & mine);
                if (lo < hi) {
                    if (cm >= mid) lo = mid;
                    else hi = mid - 1;
                }
            }
            // lane y of the group: the result of its row, when it has entries
            const uint32_t y = lane - x;
            const uint32_t yp = __shfl(ends, (y - 1) & 63, 64), ye = __shfl(ends, y & 63, 64);
            const uint32_t yb = y ? yp : 0u;
            const uint32_t nh = __shfl(lo, yb & 63, 64);
            if (lane >= x && y < cnt && ye > yb) h = nh;
        },
        [&](uint32_t x, uint32_t b, uint32_t d, const uint32_t (&e)[kRegPieces]) {
            if (d >= shared) return;
            const uint32_t H = __builtin_amdgcn_readlane(h, x);
            uint32_t lo, hi = H - 1, c = 0;
            if (d <= kRegRow) {
                uint32_t v[2 * kRegPieces];
                row_values(s_h, e, d, lane, v);
                c = count_at_least(v, d, H);
                if (c >= H) return;
                lo = c > k0 ? c : k0;
                if (lo > hi) lo = hi;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi + 1) >> 1;
                    if (count_at_least(v, d, mid) >= mid) lo = mid;
                    else hi = mid - 1;
                }
            } else {
                row_stretches(lcol, s_h, b, d, lane, e, [&](const uint32_t (&v)[2 * kRegPieces], uint32_t left) {
                    c += count_at_least(v, left, H);
                    return c < H;
                });
                if (c >= H) return;
                // a longer row is read once more, for a few thresholds below H: its bound falls below the
                // smallest one that it misses (an upper bound still; the next phases go on from there)
                constexpr uint32_t kOff[8] = {1, 2, 4, 8, 16, 64, 256, 1024};
                uint32_t n[8] = {0, 0, 0, 0, 0, 0, 0, 0};
                row_stretches(lcol, s_h, b, d, lane, e, [&](const uint32_t (&v)[2 * kRegPieces], uint32_t left) {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        if (H > kOff[q] && H - kOff[q] > k0) n[q] += count_at_least(v, left, H - kOff[q]);
                    return true;
                });
                lo = H - 1;
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (H > kOff[q] && H - kOff[q] > k0 && n[q] < H - kOff[q]) lo = H - kOff[q] - 1;
            }
            if (lane == x) h = lo;
        });
    return h;
}

// the first vertex v <= R whose work before it, lrow[v] + kVertexCost * v, is at least x (64 probes at
// a time)
__device__ __forceinline__ uint32_t split_vertex(const uint32_t *__restrict__ lrow, uint32_t R, uint64_t x, unsigned lane) {
    uint32_t lo = 0, len = R;   // the answer is in [lo, lo + len]
    while (len > 0) {
        const uint32_t step = (len + 63) / 64, i = lo + lane * step;
        const bool below = lane * step < len && (uint64_t)lrow[i < R ? i : R] + (uint64_t)kVertexCost * i < x;
        const uint32_t c = (uint32_t)__popcll(__ballot(below));   // (a prefix of the lanes)
        if (c == 0) return lo;
        const uint32_t nlo = lo + (c - 1) * step + 1, nend = lo + c * step < lo + len ? lo + c * step : lo + len;
        lo = nlo;
        len = nend - nlo;
    }
    return lo;
}

__global__ void __launch_bounds__(kBlock)
k_peel_finish(FinArgs A) {
    __shared__ __attribute__((aligned(16))) uint16_t s_v[kTail];
    __shared__ uint32_t s_key[kSlots], s_cnt[kSlots];
    __shared__ unsigned s_any, s_more, s_err, s_scan[kBlock / 64];
    __shared__ uint32_t s_row[kSharedRows], s_rows, s_ge[kSharedRows], s_at[3][8];
    PeelCtl *ctl = A.ctl;
    if (!ctl->ho || ctl->error) return;
    constexpr uint32_t kBW = kBlock / 64;
    const uint32_t R = (uint32_t)ctl->lres, k0 = ctl->ho_k, qbase = ctl->ho_tail;
    uint32_t nblk = R <= kFinSmall ? 1u : (R + kPerWave * kBW - 1) / (kPerWave * kBW);
    if (nblk > gridDim.x) nblk = gridDim.x;
    if (blockIdx.x >= nblk) return;
    const unsigned tid = threadIdx.x, lane = tid & 63;
    const uint32_t W = nblk * kBW, gw = blockIdx.x * kBW + tid / 64;
    const uint32_t gtid = blockIdx.x * kBlock + tid, gsize = nblk * kBlock;
    BarTurn turn;
    // this wavefront's vertices
    const uint64_t work = (uint64_t)A.lrow[R] + (uint64_t)kVertexCost * R;
    const uint32_t va = split_vertex(A.lrow, R, work * gw / W, lane);
    const uint32_t vb = gw + 1 < W ? split_vertex(A.lrow, R, work * (gw + 1) / W, lane) : R;
    auto group_rows = [&](uint32_t v) {
        GroupRows G;
        G.nv = vb - v < kGroup ? vb - v : kGroup;
        G.rows = A.lrow[v + (lane < G.nv ? lane : G.nv)];
        return G;
    };
    const GroupRows G0 = group_rows(va < vb ? va : (vb < R ? vb : R));
    // bounds: the degrees; no position taken
    const uint32_t cell_cap = FinishRoom::cells(R);
    // rows of twice a wavefront's share and more, which one wavefront would hold the others up with
    // (fewer than nine can begin in a block's share)
    const uint64_t share = work / nblk;
    const uint32_t shared = share / 8 > 2 * kRegRow ? (uint32_t)(share / 8) : 2 * kRegRow;
    if (tid == 0) s_rows = 0;
    if (tid < 24) s_at[tid / 8][tid % 8] = 0;
    __syncthreads();
    for (uint32_t v = va + lane; R > shared && v < vb; v += 64)
        if (A.lrow[v + 1] - A.lrow[v] >= shared) {
            const uint32_t x = atomicAdd(&s_rows, 1u);
            if (x < kSharedRows) s_row[x] = v;
            else atomicOr(&ctl->error, 64u);
        }
    for (uint32_t v = gtid; v < R; v += gsize) {
        A.val[v] = (uint16_t)(A.lrow[v + 1] - A.lrow[v]);
        A.when[v] = 0;
    }
    for (uint32_t c = gtid; c < cell_cap; c += gsize) A.cur[c] = 0;
    fin_barrier(A, nblk, turn, &s_err);
    auto load_values = [&](const uint16_t *from) {
        const uint4 *src = reinterpret_cast<const uint4 *>(from);
        uint4 *dst = reinterpret_cast<uint4 *>(s_v);
        for (uint32_t i = tid; i < (R + 7) / 8; i += kBlock) dst[i] = src[i];
        if (tid == 0) s_any = 0;
        if (tid < kSharedRows) s_ge[tid] = 0;
    };
    // the block's rows that its wavefronts walk together: f(values, entries left) for this wavefront's
    // stretches of the row at b, the first of them the one after `at` others
    auto shared_stretches = [&](uint32_t b, uint32_t d, uint32_t at, auto f) {
        for (uint32_t j = ((tid / 64 - at) % kBW) * kRegRow; j < d; j += kBW * kRegRow) {
            uint32_t c[kRegPieces], v[2 * kRegPieces];
            row_entries(A.lcol, b + j, d - j, lane, c);
            row_values(s_v, c, d - j, lane, v);
            f(v, d - j);
        }
    };
    // New bounds of those rows, exact ones: the values of at least the present bound for all of them at
    // once, then eight thresholds a pass for those that fall.  Returns how many did (to the first
    // wavefront).  A wavefront a row, some thresholds a phase, took 130 us a phase beside a row of 46,544
    // entries (200,000 vertices, 2M pairs: the peel 9.5 ms in 66 phases, 3.3 in 49 so).
    uint32_t pass = 0;
    auto shared_rows = [&](uint16_t *out, uint32_t ph) {
        const uint32_t n_rows = s_rows;
        uint32_t fell = 0, at = 0;
        for (uint32_t x = 0; x < n_rows; ++x) {
            const uint32_t v = s_row[x], b = A.lrow[v], d = A.lrow[v + 1] - b, H = s_v[v];
            uint32_t n = 0;
            shared_stretches(b, d, at, [&](const uint32_t (&w)[2 * kRegPieces], uint32_t left) {
                n += count_at_least(w, left, H);
            });
            if (lane == 0 && n) atomicAdd(&s_ge[x], n);
            at += (d + kRegRow - 1) / kRegRow;
        }
        __syncthreads();
        for (uint32_t x = 0; x < n_rows; ++x) {
            const uint32_t v = s_row[x], b = A.lrow[v], d = A.lrow[v + 1] - b, H = s_v[v], c = s_ge[x];
            if (c >= H) continue;
            uint32_t hi = H - 1, lo = c > k0 ? c : k0;
            if (lo > hi) lo = hi;
            while (lo < hi) {
                uint32_t t[8], n[8];
#pragma unroll
                for (uint32_t q = 0; q < 8; ++q) {
                    t[q] = lo + ((hi - lo) * (q + 1) + 7) / 8;
                    n[q] = 0;
                }
                shared_stretches(b, d, 0, [&](const uint32_t (&w)[2 * kRegPieces], uint32_t left) {
#pragma unroll
                    for (uint32_t q = 0; q < 8; ++q) n[q] += count_at_least(w, left, t[q]);
                });
#pragma unroll
                for (uint32_t q = 0; q < 8; ++q)
                    if (lane == 0 && n[q]) atomicAdd(&s_at[pass % 3][q], n[q]);
                __syncthreads();
#pragma unroll
                for (uint32_t q = 0; q < 8; ++q) {   // (t and the counts against it: true, then false)
                    if (s_at[pass % 3][q] >= t[q]) {
                        lo = t[q];
                    } else {
                        hi = t[q] - 1;
                        break;
                    }
                }
                // (for the pass after next: every thread has read it, and adds to it after a barrier)
                if (tid < 8) s_at[(pass + 2) % 3][tid] = 0;
                ++pass;
            }
            if (tid == 0) {
                out[v] = (uint16_t)lo;
                A.when[v] = ph + 1;
            }
            ++fell;
        }
        return tid / 64 ? 0u : fell;
    };
    // Every block learns whether a bound fell in phase ph, and every kTellPhases phases how many did: then
    // each block leaves its falls in a slot and adds up all slots (an atomic on one counter by each would take
    // as long as the barrier; adding up the slots in every phase made the finish of 61M edges 2% longer).
    auto all_fell = [&](uint32_t fell, uint32_t ph) {
        if (fell && lane == 0) atomicAdd(&s_any, fell);
        __syncthreads();
        const bool tell = ph % kTellPhases == 0;
        uint32_t *falls = A.falls + (ph / kTellPhases & 1) * FinishRoom::kBlocks;
        if (tid == 0) {
            if (tell)
                __hip_atomic_store(&falls[blockIdx.x], s_any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else if (s_any)
                __hip_atomic_store(&ctl->fin[ph % 3], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_more = 0;
        }
        group_barrier(A.bar, &ctl->error, nblk, turn);
        if (tid == kBlock - 1) s_err = ld_relaxed(&ctl->error);   // (beside the first wavefront's load)
        if (tell) {
            uint32_t n = tid < nblk ? ld_relaxed(&falls[tid]) : 0u;
            if (tid / 64 * 64 < nblk) {
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
                if (lane == 0 && n) atomicAdd(&s_more, n);
            }
        } else if (tid == 0) {
            s_more = ld_relaxed(&ctl->fin[ph % 3]);
        }
        __syncthreads();
        const uint32_t more = s_more;
        // read by every block before the next barrier: cleared for the phase after next
        if (gtid == 0)
            __hip_atomic_store(&ctl->fin[(ph + 2) % 3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return more;
    };
    // core numbers
    uint32_t ph = 0, first_fell = 0, few = 0, few_first = 0;
    for (;; ++ph) {
        load_values(A.val + (ph & 1 ? kTail : 0));
        __syncthreads();
        uint16_t *out = A.val + (ph & 1 ? 0 : kTail);
        uint32_t fell = 0;   // of this wavefront
        for (uint32_t v0 = va; v0 < vb; v0 += kGroup) {
            const GroupRows G = v0 == va ? G0 : group_rows(v0);
            const uint32_t v = v0 + lane;
            const uint32_t h = lane < G.nv ? s_v[v] : 0u;
            const uint32_t nh = group_bounds(G, A.lcol, s_v, h, k0, shared, lane);
            if (lane < G.nv) {
                out[v] = (uint16_t)nh;
                if (nh != h) A.when[v] = ph + 1;
            }
            fell += (uint32_t)__popcll(__ballot(lane < G.nv && nh != h));
        }
        if (s_rows) {
            __syncthreads();   // (the wavefronts' own bounds written)
            fell += shared_rows(out, ph);
        }
        const uint32_t more = all_fell(fell, ph);
        if (s_err) return;
        if (!more) break;
        bool leave = ph + 1 >= kPhaseMost;
        if (ph % kTellPhases == 0) {
            if (ph == 0) first_fell = more;
            if (more > kFewFell || more > 2 * few_first) few = 0;
            if (few == 0) few_first = more;
            few += more <= kFewFell ? 1 : 0;
            leave |= (ph == kSlowPhase && 4 * more > first_fell) || few > kFewPhases / kTellPhases;
        }
        if (leave) {
            if (gtid == 0) ctl->left = 1;   // (every block sees the same counts, and leaves)
            return;
        }
    }
    // s_v holds the core numbers (nothing fell in this last phase ph); the largest of them
    if (tid == 0) s_any = 0;
    __syncthreads();
    uint32_t top = 0;
    for (uint32_t v = tid; v < R; v += kBlock) top = s_v[v] > top ? s_v[v] : top;
    if (top) atomicMax(&s_any, top);
    __syncthreads();
    const uint32_t kmax = s_any;
    const uint32_t T = ph + 1, shells = kmax >= k0 ? kmax - k0 + 1 : 1;
    constexpr uint32_t kCls = FinishRoom::kClasses;
    const bool wide = (uint64_t)shells * T * kCls > cell_cap;   // cells beyond the room for them
    const uint32_t cells = wide ? (shells < cell_cap ? shells : cell_cap) : shells * T * kCls;
    // this block's vertices, one a thread and chunk: their places among those of their cell, taken with
    // one atomic a block, chunk and cell where the cell's slot in LDS is free for it.  Beyond the room the
    // cells are the shells, and the phases take their places one after the other.
    const uint32_t ba = blockIdx.x, first = split_vertex(A.lrow, R, work * (ba * kBW) / W, lane);
    const uint32_t last = ba + 1 < nblk ? split_vertex(A.lrow, R, work * ((ba + 1) * kBW) / W, lane) : R;
    auto cell_of = [&](uint32_t v) {
        const uint32_t c = s_v[v] > k0 ? s_v[v] - k0 : 0u;
        return wide ? c : (c * T + A.when[v]) * kCls + FinishRoom::deg_class(A.lrow[v + 1] - A.lrow[v], s_v[v]);
    };
    for (uint32_t t = 0; t < (wide ? T : 1u); ++t) {
        for (uint32_t v0 = first; v0 < last; v0 += kBlock) {
            for (uint32_t x = tid; x < kSlots; x += kBlock) {
                s_key[x] = ~0u;
                s_cnt[x] = 0;
            }
            __syncthreads();
            const uint32_t v = v0 + tid;
            const bool in = v < last && (!wide || A.when[v] == t);
            const uint32_t cell = in ? cell_of(v) : 0u, slot = cell % kSlots;
            if (in && !wide) A.when[v] = cell;   // (this thread's own from here on)
            uint32_t at = 0;
            bool held = false;
            if (in) {
                const uint32_t was = atomicCAS(&s_key[slot], ~0u, cell);
                held = was == ~0u || was == cell;
                at = held ? atomicAdd(&s_cnt[slot], 1u) : atomicAdd(&A.cur[cell], 1u);
            }
            __syncthreads();
            for (uint32_t x = tid; x < kSlots; x += kBlock)
                if (s_cnt[x]) s_cnt[x] = atomicAdd(&A.cur[s_key[x]], s_cnt[x]);
            __syncthreads();
            if (in) A.pos[v] = held ? s_cnt[slot] + at : at;
            __syncthreads();
        }
        fin_barrier(A, nblk, turn, &s_err);
        if (s_err) return;
    }
    // first position of every cell that holds a vertex: every block writes the same ones, and reads its own
    // back
    constexpr uint32_t kPer = 8;   // cells a thread
    uint32_t run = 0;
    for (uint32_t c0 = 0; c0 < cells && run < R; c0 += kPer * kBlock) {
        const uint32_t c = c0 + kPer * tid;
        uint32_t n[kPer], mine = 0;
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
            n[j] = c + j < cells ? A.cur[c + j] : 0u;
            mine += n[j];
        }
        uint32_t x = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= (unsigned)o) x += y;
        }
        if (lane == 63) s_scan[tid / 64] = x;
        __syncthreads();
        uint32_t before = 0, total = 0;
        for (uint32_t w = 0; w < kBW; ++w) {
            before += w < tid / 64 ? s_scan[w] : 0u;
            total += s_scan[w];
        }
        uint32_t at = run + before + x - mine;
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
            if (n[j]) A.base[c + j] = at;
            at += n[j];
        }
        run += total;
        __syncthreads();
    }
    // positions and core numbers, each by the lane that took the position
    for (uint32_t v0 = first; v0 < last; v0 += kBlock) {
        const uint32_t v = v0 + tid;
        if (v < last) {
            const uint32_t p = qbase + A.base[wide ? cell_of(v) : A.when[v]] + A.pos[v], x = A.rlist[v];
            if (p < qbase + R) A.queue[p] = x;
            else atomicOr(&ctl->error, 16u);
            A.level[x] = s_v[v];
        }
    }
    if (gtid == 0) {
        ctl->kappa = kmax > k0 ? kmax : k0;
        ctl->rounds = ctl->ho_rounds + T;
        __hip_atomic_store(&ctl->qtail, qbase + R, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ------------------------------------------------------------------------------------------------
// The levels of the vertices that the finish leaves: where a fall travels one vertex a phase (long chains,
// lattices), a phase a hop, each with a grid barrier and every row, costs far more than a removal round of
// a workgroup.  One workgroup takes the last vertices, level by level, on the subgraph they induce, with
// local (16-bit) vertex ids.  The local CSR rows, the degrees, the removal queue and the list of vertices
// not yet queued live in LDS, so a round touches global memory only to read adjacency (lcol);
// workgroup barriers separate rounds.  rlist maps local ids to vertices.  A degree counts the
// neighbours not yet removed (so it never falls below zero, and two 16-bit degrees share a word
// safely) until the vertex is queued; queuing adds kMark - degree, which puts it at kMark, and
// the at most kLevelTail later decrements leave it at least kMark - kLevelTail, above every level.  Each
// wavefront keeps its own segment of the live list and compacts it in place at every level scan,
// so a scan reads only the vertices still live, and takes one atomic per wavefront for the
// survivors' count and smallest degree.  The queue positions (continuing from qbase) and the core
// numbers are written at the end, from the queue and the level boundaries recorded in lvl (pairs:
// first queue position, level).  A path of 16,000 vertices: 46.7 ms by phases, 6.1 so.
// ------------------------------------------------------------------------------------------------
constexpr uint32_t kLevelTail = kPeelTailMax;   // most vertices of it: what one workgroup's LDS holds
constexpr uint32_t kRowWords = kLevelTail + 1, kDegWords = kLevelTail / 2, kQWords = kLevelTail / 2,
                   kLiveWords = kLevelTail / 2;
constexpr uint32_t kMark = 0xC000u, kMarked = 0x8000u;
static_assert(kMark - kLevelTail > kMarked && kMarked > kLevelTail, "queued degrees stay above every level");
__global__ void __launch_bounds__(kBlock)
k_peel_levels(const uint32_t *__restrict__ rlist, const uint32_t *__restrict__ lrow, const uint16_t *__restrict__ lcol,
              uint32_t *__restrict__ lvl, uint32_t *__restrict__ level, uint32_t *__restrict__ queue,
              PeelCtl *__restrict__ ctl) {
    __shared__ __attribute__((aligned(16))) uint32_t s_mem[kRowWords + kDegWords + kQWords + kLiveWords];
    if (!ctl->ho || ctl->error) return;
    const uint32_t R = (uint32_t)ctl->lres, qbase = ctl->ho_tail;
    uint32_t k = ctl->ho_k, rounds = ctl->ho_rounds;
    uint32_t *s_row = s_mem;                                              // kRowWords
    uint32_t *s_deg = s_mem + kRowWords;                                  // kDegWords
    uint16_t *s_q = reinterpret_cast<uint16_t *>(s_mem + kRowWords + kDegWords);               // kLevelTail
    uint16_t *s_live = reinterpret_cast<uint16_t *>(s_mem + kRowWords + kDegWords + kQWords);  // kLevelTail
    __shared__ unsigned s_qt, s_keep, s_min, s_nlvl;
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid / 64;
    constexpr unsigned kWaves = kBlock / 64;
    const uint64_t below = (1ull << lane) - 1;
    for (uint32_t l = tid; l <= R; l += kBlock) s_row[l] = lrow[l];
    for (uint32_t w = tid; w < kDegWords; w += kBlock) s_deg[w] = 0;
    for (uint32_t l = tid; l < R; l += kBlock) s_live[l] = (uint16_t)l;
    __syncthreads();
    for (uint32_t l = tid; l < R; l += kBlock)
        atomicAdd(&s_deg[l >> 1], (s_row[l + 1] - s_row[l]) << ((l & 1) * 16));
    if (tid == 0) {
        s_qt = 0;
        s_nlvl = 0;
    }
    // this wavefront's segment of the live list: [lb, lb + lc)
    const uint32_t seg = (R + kWaves - 1) / kWaves;
    const uint32_t lb = wave * seg < R ? wave * seg : R;
    uint32_t lc = (lb + seg < R ? lb + seg : R) - lb;
    uint32_t h = 0, t = 0;
    auto deg_of = [&](uint32_t l) { return (s_deg[l >> 1] >> ((l & 1) * 16)) & 0xffffu; };
    // queue y, whose degree is d (no decrement of y runs between reading d and this)
    auto mark = [&](uint32_t y, uint32_t d) { atomicAdd(&s_deg[y >> 1], (kMark - d) << ((y & 1) * 16)); };
    // remove one edge end at y; a degree taken from k + 1 to k queues y
    auto dec = [&](uint32_t y, uint32_t kk) {
        const uint32_t sh = (y & 1) * 16;
        const uint32_t old = (atomicSub(&s_deg[y >> 1], 1u << sh) >> sh) & 0xffffu;
        if (old == kk + 1) {
            atomicAdd(&s_deg[y >> 1], (kMark - kk) << sh);
            const uint32_t p = atomicAdd(&s_qt, 1u);
            if (p < R) s_q[p] = (uint16_t)y;
        }
    };
    while (true) {
        __syncthreads();
        if (tid == 0) {
            s_keep = 0;
            s_min = 0xffffffffu;
        }
        __syncthreads();
        const uint32_t level_start = t;
        // level scan over this wavefront's live vertices: queue those of degree <= k, keep the
        // others (written back in place: a survivor's new slot is never after its old one, and
        // the wavefront reads a chunk before it writes any of it)
        {
            uint32_t nk = 0;
            unsigned md = 0xffffffffu;
            for (uint32_t i0 = 0; i0 < lc; i0 += 64) {
                const uint32_t i = i0 + lane;
                uint32_t l = 0, d = kMark;
                if (i < lc) {
                    l = s_live[lb + i];
                    d = deg_of(l);
                }
                const bool tk = d <= k, kp = d > k && d < kMarked;
                const uint64_t mt = __ballot(tk), mk = __ballot(kp);
                if (mt) {
                    uint32_t qb = 0;
                    if (lane == 0) qb = atomicAdd(&s_qt, (unsigned)__popcll(mt));
                    qb = __shfl(qb, 0, 64);
                    if (tk) {
                        const uint32_t p = qb + (uint32_t)__popcll(mt & below);
                        mark(l, d);
                        if (p < R) s_q[p] = (uint16_t)l;
                    }
                }
                if (kp) {
                    s_live[lb + nk + (uint32_t)__popcll(mk & below)] = (uint16_t)l;
                    md = d < md ? d : md;
                }
                nk += (uint32_t)__popcll(mk);
            }
            lc = nk;
            md = wave_min(md);
            if (lane == 0 && nk) {
                atomicAdd(&s_keep, nk);
                atomicMin(&s_min, md);
            }
        }
        __syncthreads();
        t = s_qt;
        const uint32_t keep = s_keep, md = s_min;
        if (keep == 0) h = t;   // every remaining vertex is queued: nothing left to update
        // rounds: remove s_q[h, t)
        while (h < t) {
            const uint32_t f = t - h;
            uint32_t i0, first, stride, step;
            if (f >= kWaves) {
                i0 = h + wave; first = lane; stride = 64; step = kWaves;
            } else {
                const uint32_t per = kWaves / f;
                i0 = h + wave / per; first = (wave % per) * 64 + lane; stride = per * 64; step = f;
                if (wave / per >= f) i0 = t;
            }
            for (uint32_t i = i0; i < t; i += step) {
                const uint32_t x = s_q[i];
                const uint32_t e = s_row[x + 1];
                uint32_t j = s_row[x] + first;
                for (; j + 3 * stride < e; j += 4 * stride) {
                    const uint32_t y0 = lcol[j], y1 = lcol[j + stride], y2 = lcol[j + 2 * stride],
                                   y3 = lcol[j + 3 * stride];
                    dec(y0, k);
                    dec(y1, k);
                    dec(y2, k);
                    dec(y3, k);
                }
                for (; j < e; j += stride) dec(lcol[j], k);
            }
            ++rounds;
            __syncthreads();
            h = t;
            t = s_qt;
            __syncthreads();
        }
        if (t > level_start && tid == 0) {   // this level removed s_q[level_start, t)
            const uint32_t li = s_nlvl++;
            lvl[2 * li] = level_start;
            lvl[2 * li + 1] = k;
        }
        if (t >= R) break;
        uint32_t next = k + 1;
        if (t == level_start && md != 0xffffffffu && md > next) next = md;
        k = next;
        if (k > R + qbase + 1) {   // cannot happen, as in the grid loop
            if (tid == 0) atomicOr(&ctl->error, 2u);
            break;
        }
    }
    __syncthreads();
    // queue positions and core numbers of the removed vertices, in removal order
    const uint32_t nl = s_nlvl, nq = t < R ? t : R;
    __threadfence_block();
    for (uint32_t p = tid; p < nq; p += kBlock) {
        const uint32_t v = rlist[s_q[p]];
        queue[qbase + p] = v;
        uint32_t lo = 0, len = nl;   // last boundary at or before p
        while (len > 0) {
            const uint32_t half = len >> 1;
            if (lvl[2 * (lo + half)] <= p) {
                lo += half + 1;
                len -= half + 1;
            } else {
                len = half;
            }
        }
        level[v] = lo > 0 ? lvl[2 * (lo - 1) + 1] : k;
    }
    if (tid == 0) {
        __hip_atomic_store(&ctl->qtail, qbase + nq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ctl->kappa = k;
        ctl->rounds = rounds;
        ctl->left = 0;
    }
}

// Where the level peel begins: with the whole graph, or (left > 0) with the vertices rlist[0, left) that
// the finish left to it, at level k, with `tail` positions taken.
struct PeelStart {
    uint32_t left, k, tail, rounds;
};

__global__ void __launch_bounds__(kBlock)
k_peel(PeelStart from, uint32_t n, const uint32_t *__restrict__ row, const uint32_t *__restrict__ col,
       int *__restrict__ deg, uint32_t *__restrict__ level, uint32_t *__restrict__ queue,
       uint32_t *__restrict__ alive_a, uint32_t *__restrict__ alive_b, uint32_t *__restrict__ loc,
       uint32_t *__restrict__ rlist, uint32_t *__restrict__ lrow, uint64_t lcol_cap, uint32_t tail_cap,
       uint32_t *__restrict__ ovf0,
       uint32_t *__restrict__ ovf1, PeelCtl *__restrict__ ctl, unsigned *__restrict__ bar) {
    // the whole grid takes part while many vertices remain, then ever fewer of its first blocks
    unsigned nblk = gridDim.x;
    const uint32_t gtid = blockIdx.x * kBlock + threadIdx.x;
    uint32_t gsize = nblk * kBlock;
    const uint32_t gwave = gtid / 64, lane = threadIdx.x & 63;
    uint32_t nwaves = gsize / 64;
    const uint64_t below = (1ull << lane) - 1;
    BarTurn turn;
    __shared__ __attribute__((aligned(16))) uint32_t s_mem[kLdsWords];
    __shared__ unsigned s_cnt, s_base;
    __shared__ unsigned s_wct[kBlock / 64], s_wck[kBlock / 64], s_wmd[kBlock / 64], s_bq, s_bk;

    // the host cleared the control block; initialise per-vertex state
    for (uint32_t i = gtid; i < from.left; i += gsize) {
        const uint32_t v = rlist[i];
        alive_a[i] = v;
        loc[v] = kUnset;
    }
    for (uint32_t v = gtid; !from.left && v < n; v += gsize) {
        deg[v] = (int)(row[v + 1] - row[v]);
        level[v] = kUnset;
        alive_a[v] = v;
        loc[v] = kUnset;
        queue[v] = kUnset;   // (a place that nothing takes is found with the ranks)
    }
    if (gtid == 0)
        for (int x = 0; x < 3; ++x) ctl->scan[x][1] = 0xffffffffu;
    group_barrier(bar, &ctl->error, nblk, turn);

    // tail: vertices queued before the current grid phase (a scan or a round); phase ph takes its
    // queue positions tail + [0, qc[ph % 3]) and every block adds the final count after the phase's
    // barrier, so all blocks agree on tail although a fast block may already be in the next phase
    uint32_t k = from.k, head = from.tail, tail = from.tail, n_alive = from.left ? from.left : n, prev_tail = from.tail,
             rounds = from.rounds, lv = 0, ph = 0;
    uint32_t *cur = alive_a, *nxt = alive_b;
    bool done = false;
    // here every queued vertex has been removed: n - tail vertices remain
    while (n - tail > tail_cap) {
        // level scan: queue every remaining vertex of degree <= k, keep the others.  Each
        // wavefront takes a contiguous segment and counts its picks and survivors; its block
        // reserves room for all of them in both lists (one atomic each), and each wavefront then
        // writes its picks in order (no degree changes during a scan), so both lists keep the
        // roughly ascending vertex order of the previous one and the degree reads of the next scan
        // stay coalesced.
        {
            const uint32_t seg = ((n_alive + nwaves - 1) / nwaves + 63) & ~63u;
            const uint32_t sb = gwave * seg < n_alive ? gwave * seg : n_alive;
            const uint32_t se = sb + seg < n_alive ? sb + seg : n_alive;
            uint32_t ct = 0, ck = 0;
            unsigned mdl = 0xffffffffu;
            // four chunks of 64 at a time: their list reads, then their degree reads, in flight
            // together
            for (uint32_t b0 = sb; b0 < se; b0 += 4 * 64) {
                uint32_t vv[4];
                int dd[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t i = b0 + q * 64 + lane;
                    vv[q] = i < se ? cur[i] : 0u;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    dd[q] = b0 + q * 64 + lane < se ? ld_relaxed(&deg[vv[q]]) : -1;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int d = dd[q];
                    const bool keep = d > (int)k;
                    ct += (uint32_t)__popcll(__ballot(d >= 0 && d <= (int)k));   // d < 0: queued
                    ck += (uint32_t)__popcll(__ballot(keep));
                    mdl = keep && (unsigned)d < mdl ? (unsigned)d : mdl;
                }
            }
            mdl = wave_min(mdl);
            // one reservation per block (the wavefronts' segments are consecutive, so a prefix
            // over them keeps the order): thousands of wavefronts meeting at the same counters
            // would serialise there
            const unsigned wv = threadIdx.x / 64;
            if (lane == 0) {
                s_wct[wv] = ct;
                s_wck[wv] = ck;
                s_wmd[wv] = mdl;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                unsigned tct = 0, tck = 0, bmd = 0xffffffffu;
                for (unsigned w = 0; w < kBlock / 64; ++w) {
                    const unsigned a = s_wct[w], b = s_wck[w];
                    s_wct[w] = tct;
                    s_wck[w] = tck;
                    tct += a;
                    tck += b;
                    bmd = s_wmd[w] < bmd ? s_wmd[w] : bmd;
                }
                s_bq = tct ? tail + atomicAdd(&ctl->qc[ph % 3], tct) : 0u;
                s_bk = tck ? atomicAdd(&ctl->scan[lv % 3][0], tck) : 0u;
                if (bmd != 0xffffffffu) atomicMin(&ctl->scan[lv % 3][1], bmd);
            }
            __syncthreads();
            uint32_t qb = s_bq + s_wct[wv], kb = s_bk + s_wck[wv];
            if (ct | ck) {
                for (uint32_t b0 = sb; b0 < se; b0 += 4 * 64) {
                    uint32_t vv[4];
                    int dd[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t i = b0 + q * 64 + lane;
                        vv[q] = i < se ? cur[i] : 0u;
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dd[q] = b0 + q * 64 + lane < se ? ld_relaxed(&deg[vv[q]]) : -1;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t v = vv[q];
                        const int d = dd[q];
                        const bool take = d >= 0 && d <= (int)k, keep = d > (int)k;
                        const uint64_t mt = __ballot(take), mk = __ballot(keep);
                        if (take) {
                            level[v] = k;
                            const uint32_t p = qb + (uint32_t)__popcll(mt & below);
                            if (p < n) queue[p] = v;
                        }
                        if (keep) nxt[kb + (uint32_t)__popcll(mk & below)] = v;
                        qb += (uint32_t)__popcll(mt);
                        kb += (uint32_t)__popcll(mk);
                    }
                }
            }
        }
        group_barrier(bar, &ctl->error, nblk, turn);
        tail += ld_relaxed(&ctl->qc[ph % 3]);
        const uint32_t na2 = ld_relaxed(&ctl->scan[lv % 3][0]), md = ld_relaxed(&ctl->scan[lv % 3][1]);
        // the counters of the previous level were read by every block before this barrier: clear
        // them for the level after next (the next level's barrier publishes the clearing)
        if (gtid == 0) {
            __hip_atomic_store(&ctl->scan[(lv + 2) % 3][0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->scan[(lv + 2) % 3][1], 0xffffffffu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->qc[(ph + 2) % 3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ctl->ovc[(ph + 2) % 3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        ++lv;
        ++ph;
        // few vertices left: the later levels are latency-bound, and a barrier costs more the
        // more blocks meet at it, so the grid narrows in steps (only ever narrows)
        {
            unsigned want = kWidths[2].blocks;
            for (const Width &w : kWidths)
                if (na2 >= w.from || n_alive - na2 >= kBusy) {
                    want = w.blocks;
                    break;
                }
            if (want < nblk) {
                if (blockIdx.x >= want) return;
                nblk = want;
                gsize = nblk * kBlock;
                nwaves = gsize / 64;
            }
        }
        // no survivors: every remaining vertex is queued at this level, and removing them can
        // queue nothing more
        if (na2 == 0) head = tail;
        // Rounds.  The frontier of the first is the scan's picks, queue[head, tail); each block
        // removes its share and then, without a grid barrier, removes the vertices that its own
        // removals queued (its staging list), step after step, until it queues nothing more; those
        // take their queue positions when their removal starts.  Only vertices queued past a full
        // staging list wait for the next round (overflow list; their positions are the round's
        // first).  A frontier of at least one vertex per wavefront is split by vertex; a smaller one
        // gives each vertex an equal share of the wavefronts.
        // Any order of removal within a level is a degeneracy ordering as long as every vertex
        // takes its position no later than its removal starts: a neighbour placed after it was not
        // yet removed when it was queued, so it counts among the at most k neighbours it had then.
        {
            uint32_t nf = tail - head;
            const uint32_t *fl = queue + head;
            bool first = true;
            while (nf > 0) {
                uint32_t *ovf_out = (ph & 1) ? ovf1 : ovf0;
                unsigned *ovc = &ctl->ovc[ph % 3];
                const uint32_t qbase = first ? tail : tail + nf;
                if (!first)
                    for (uint32_t i = gtid; i < nf; i += gsize)
                        if (tail + i < n) queue[tail + i] = fl[i];
                uint32_t *stage = s_mem, *front = s_mem + kStage;
                if (threadIdx.x == 0) s_cnt = 0;
                __syncthreads();
                if (nf >= nwaves) {
                    for (uint32_t i = gwave; i < nf; i += nwaves)
                        remove_edges(fl[i], lane, 64, k, n, row, col, deg, level, ovc, ovf_out, &ctl->error,
                                     stage, &s_cnt);
                } else {
                    const uint32_t per = nwaves / nf;
                    const uint32_t i = gwave / per, sub = gwave % per;
                    if (i < nf)
                        remove_edges(fl[i], sub * 64 + lane, per * 64, k, n, row, col, deg, level, ovc, ovf_out,
                                     &ctl->error, stage, &s_cnt);
                }
                // the block's own cascade
                for (uint32_t steps = 0;; ++steps) {
                    __syncthreads();
                    const uint32_t c = s_cnt < kStage ? s_cnt : kStage;
                    if (c == 0 || steps > n) break;
                    __syncthreads();
                    if (threadIdx.x == 0) {
                        s_base = qbase + atomicAdd(&ctl->qc[ph % 3], c);
                        s_cnt = 0;
                    }
                    uint32_t *t = stage;
                    stage = front;
                    front = t;
                    // this wavefront's first vertex and its adjacency bounds, read while the
                    // positions are being taken (reads only: its removal starts after them)
                    constexpr uint32_t kBW = kBlock / 64;
                    const uint32_t wave = threadIdx.x / 64;
                    const uint32_t per = c >= kBW ? 1 : kBW / c;
                    const uint32_t i0 = wave / per, sub = wave % per;
                    uint32_t rb = 0, re = 0;
                    if (i0 < c) {
                        const uint32_t v0 = front[i0];
                        rb = row[v0];
                        re = row[v0 + 1];
                    }
                    __syncthreads();
                    for (uint32_t x = threadIdx.x; x < c; x += kBlock) {
                        const uint32_t p = s_base + x;
                        if (p < n) queue[p] = front[x];
                    }
                    if (c >= kBW) {
                        if (i0 < c)
                            remove_range(rb, re, lane, 64, k, n, col, deg, level, ovc, ovf_out, &ctl->error, stage,
                                         &s_cnt);
                        for (uint32_t i = i0 + kBW; i < c; i += kBW)
                            remove_edges(front[i], lane, 64, k, n, row, col, deg, level, ovc, ovf_out, &ctl->error,
                                         stage, &s_cnt);
                    } else if (i0 < c) {
                        remove_range(rb, re, sub * 64 + lane, per * 64, k, n, col, deg, level, ovc, ovf_out,
                                     &ctl->error, stage, &s_cnt);
                    }
                }
                ++rounds;
                group_barrier(bar, &ctl->error, nblk, turn);
                tail = qbase + ld_relaxed(&ctl->qc[ph % 3]);
                head = tail;
                nf = ld_relaxed(ovc);
                fl = ovf_out;
                first = false;
                if (gtid == 0) {
                    __hip_atomic_store(&ctl->qc[(ph + 2) % 3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&ctl->ovc[(ph + 2) % 3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                ++ph;
                if (nf > n) {   // cannot happen: a vertex is queued once
                    if (gtid == 0) atomicOr(&ctl->error, 8u);
                    nf = 0;
                }
            }
        }
        if (tail >= n || ld_relaxed(&ctl->error)) {
            done = true;
            break;
        }
        // every survivor now has degree > k; when this level removed nothing, no degree changed
        // since the scan, so the smallest survivor degree is the next level that removes anything
        uint32_t next = k + 1;
        if (tail == prev_tail && md != 0xffffffffu && md > next) next = md;
        prev_tail = tail;
        k = next;
        if (k > n + 1) {   // cannot happen: some vertex is removed at the smallest survivor degree
            if (gtid == 0) atomicOr(&ctl->error, 2u);
            done = true;
            break;
        }
        n_alive = na2;
        uint32_t *t = cur;
        cur = nxt;
        nxt = t;
    }
    if (done) {
        if (gtid == 0) {
            ctl->kappa = k;
            ctl->rounds = rounds;
            __hip_atomic_store(&ctl->qtail, tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    // Hand over to the finish.  Every remaining vertex is in cur with its degree (the number
    // of its remaining neighbours, since every queued vertex has been removed): give it a local
    // id and that many consecutive entries of the local adjacency (one 64-bit atomic per
    // wavefront reserves both, so rows follow local ids and lrow is a CSR row array), then write
    // its remaining neighbours' local ids there.
    for (uint32_t b0 = gwave * 64; b0 < n_alive; b0 += nwaves * 64) {
        const uint32_t i = b0 + lane;
        uint32_t v = 0;
        int d = -1;
        if (i < n_alive) {
            v = cur[i];
            d = ld_relaxed(&deg[v]);
        }
        const bool live = d >= 0;
        const uint64_t ml = __ballot(live);
        // inclusive prefix of the live degrees within the wavefront
        uint32_t inc = live ? (uint32_t)d : 0u;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, 64);
            if (lane >= (unsigned)o) inc += y;
        }
        const uint32_t tot = __shfl(inc, 63, 64);
        unsigned long long base = 0;
        if (lane == 0 && ml)
            base = atomicAdd(&ctl->lres, ((unsigned long long)tot << 32) | (unsigned long long)__popcll(ml));
        base = __shfl(base, 0, 64);
        if (live) {
            const uint32_t lid = (uint32_t)base + (uint32_t)__popcll(ml & below);
            const uint64_t off = (base >> 32) + inc - (uint32_t)d;
            if (lid < kTail && off + (uint32_t)d <= lcol_cap) {
                rlist[lid] = v;
                loc[v] = lid;
                lrow[lid] = (uint32_t)off;
            } else {
                atomicOr(&ctl->error, 4u);
            }
        }
    }
    group_barrier(bar, &ctl->error, nblk, turn);
    const unsigned long long lres = __hip_atomic_load(&ctl->lres, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t R = (uint32_t)lres, total = (uint32_t)(lres >> 32);
    if (R != n - tail || R > kTail || total > lcol_cap || ld_relaxed(&ctl->error)) {
        if (gtid == 0) atomicOr(&ctl->error, 4u);
        return;
    }
    if (gtid == 0) {
        lrow[R] = total;
        ctl->ho_tail = tail;
        ctl->ho_k = k;
        ctl->ho_rounds = rounds;
        ctl->ho = 1;
    }
}

// The hand-over's local adjacency: for every local vertex, its remaining neighbours' local ids,
// found by a scan of its whole row with one wavefront.  A launch of its own on the whole device
// (the grid has narrowed by then, and the rows of the last vertices, hubs, are long).
__global__ void __launch_bounds__(256)
k_local_adj(const uint32_t *__restrict__ row, const uint32_t *__restrict__ col, const int *__restrict__ deg,
            const uint32_t *__restrict__ loc, const uint32_t *__restrict__ rlist, const uint32_t *__restrict__ lrow,
            uint16_t *__restrict__ lcol, PeelCtl *__restrict__ ctl) {
    if (!ctl->ho || ctl->error) return;
    const uint32_t R = (uint32_t)ctl->lres;
    const unsigned lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1;
    const uint32_t nwaves = gridDim.x * (256 / 64);
    for (uint32_t l = blockIdx.x * (256 / 64) + threadIdx.x / 64; l < R; l += nwaves) {
        const uint32_t v = rlist[l], b = lrow[l];
        const uint32_t d = (uint32_t)deg[v];
        const uint32_t e = row[v + 1];
        uint32_t c = 0;
        for (uint32_t j0 = row[v]; j0 < e; j0 += 64) {
            const uint32_t j = j0 + lane;
            const uint32_t lx = j < e ? loc[col[j]] : kUnset;
            const uint64_t m = __ballot(lx != kUnset);
            const uint32_t p = c + (uint32_t)__popcll(m & below);
            if (lx != kUnset && p < d) lcol[b + p] = (uint16_t)lx;
            c += (uint32_t)__popcll(m);
        }
        if (lane == 0 && c != d) atomicOr(&ctl->error, 4u);
    }
}

// the ranks; an id that is no vertex (a place of the queue that nothing took) is an error
__global__ void k_finish(uint32_t n, const uint32_t *__restrict__ queue, uint32_t *__restrict__ rank,
                         PeelCtl *__restrict__ ctl) {
    const uint32_t p = blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const uint32_t v = queue[p];
    if (ctl->left) return;   // (not all of them ordered yet)
    if (v < n) rank[v] = p;
    else atomicOr(&ctl->error, 32u);
}

}  // namespace

int peel(dt_graph *g) {
    dt_ctx *ctx = g->ctx;
    hipStream_t st = ctx->stream;
    const uint32_t n = g->n;
    DevMem deg, alive, alive2, ctlm, loc, rlist, lrow, lcol, ovf0, ovf1, fin;
    DT_TRY(dev_alloc(ctx, deg, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, alive, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, alive2, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, ovf0, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, ovf1, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, g->core, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, g->order, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, g->rank, (uint64_t)n * 4));
    // control block, then the barrier counters of the levels and of the finish (cleared together)
    constexpr uint64_t kCtlBytes = 512, kBarBytes = kBarWords * 4;
    static_assert(sizeof(PeelCtl) <= kCtlBytes, "control block layout");
    DT_TRY(dev_alloc(ctx, ctlm, kCtlBytes + 2 * kBarBytes));
    // the finish: at most tail_cap vertices, their adjacency within 2 m_static entries and below
    // tail_cap (tail_cap - 1) as well
    const uint32_t tail_cap = g->tuning.peel_tail ? g->tuning.peel_tail : kTail;
    const uint64_t lcol_cap = std::min<uint64_t>(2ull * g->m_s, (uint64_t)tail_cap * (tail_cap - 1));
    DT_TRY(dev_alloc(ctx, loc, (uint64_t)n * 4));
    DT_TRY(dev_alloc(ctx, rlist, (uint64_t)tail_cap * 4));
    DT_TRY(dev_alloc(ctx, lrow, ((uint64_t)tail_cap + 1) * 4));
    DT_TRY(dev_alloc(ctx, fin, FinishRoom::kWords * 4));
    DT_TRY(dev_alloc(ctx, lcol, (lcol_cap + kPiece) * 2));   // (the finish reads whole pieces)
    if (n == 0) {
        g->kappa = 0;
        g->peel_rounds = 0;
        return DT_OK;
    }
    // co-resident grid (the cooperative launch fails rather than run a grid that cannot be)
    int per_cu = 0;
    DT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_peel, kBlock, 0));
    if (per_cu <= 0) return fail(DT_EDEVICE, "peel kernel cannot be resident");
    unsigned grid = kGridWide;
    if (grid > (unsigned)ctx->num_cus * (unsigned)per_cu) grid = (unsigned)ctx->num_cus * (unsigned)per_cu;
    uint32_t *level = g->core.as<uint32_t>();
    uint32_t *queue = g->order.as<uint32_t>();
    const uint32_t *row = g->row.as<uint32_t>(), *col = g->col.as<uint32_t>();
    int *degp = deg.as<int>();
    uint32_t *aa = alive.as<uint32_t>(), *ab = alive2.as<uint32_t>();
    PeelCtl *ctl = ctlm.as<PeelCtl>();
    uint32_t *locp = loc.as<uint32_t>(), *rl = rlist.as<uint32_t>(), *lb = lrow.as<uint32_t>();
    uint16_t *lc = lcol.as<uint16_t>();
    unsigned *lbar = reinterpret_cast<unsigned *>(ctlm.as<uint8_t>() + kCtlBytes);
    uint32_t *o0 = ovf0.as<uint32_t>(), *o1 = ovf1.as<uint32_t>();
    PeelCtl &h = *reinterpret_cast<PeelCtl *>(ctx->pinned_stage);
    // the levels on the grid from `from` on, until at most tcap vertices remain, and these vertices' local
    // adjacency
    auto grid_levels = [&](PeelStart from, uint32_t tcap) -> int {
        DT_HIP(hipMemsetAsync(ctlm.ptr, 0, kCtlBytes + 2 * kBarBytes, st));
        uint32_t nn = n;
        uint64_t lcap = lcol_cap;
        const unsigned blocks = std::min(grid, grid_for(from.left ? from.left : n, kBlock));
        void *args[] = {&from, &nn, &row, &col, &degp, &level, &queue, &aa, &ab, &locp, &rl, &lb, &lcap, &tcap,
                        &o0, &o1, &ctl, &lbar};
        const bool mark = !from.left;   // (levels after the finish belong to its time)
        if (mark) prof_begin(ctx, kProfPeel, st);
        DT_HIP(hipLaunchCooperativeKernel((const void *)k_peel, dim3(blocks), dim3(kBlock), args, 0, st));
        if (mark) prof_end(ctx, kProfPeel, st);
        if (mark) prof_begin(ctx, kProfPeelAdj, st);
        k_local_adj<<<(unsigned)ctx->num_cus * 8, 256, 0, st>>>(row, col, degp, locp, rl, lb, lc, ctl);
        if (mark) prof_end(ctx, kProfPeelAdj, st);
        DT_HIP(hipGetLastError());
        return DT_OK;
    };
    // the ranks (what the orientation reads next), whose check of the queue the read-back takes along
    auto ranks = [&]() -> int {
        k_finish<<<grid_for(n, 256), 256, 0, st>>>(n, queue, g->rank.as<uint32_t>(), ctl);
        DT_HIP(hipGetLastError());
        DT_HIP(hipMemcpyAsync(&h, ctl, sizeof(h), hipMemcpyDeviceToHost, st));
        DT_HIP(hipStreamSynchronize(st));
        return DT_OK;
    };
    DT_TRY(grid_levels(PeelStart{}, tail_cap));
    prof_begin(ctx, kProfPeelTail, st);
    FinArgs fa;
    fa.rlist = rl;
    fa.lrow = lb;
    fa.lcol = lc;
    fa.base = fin.as<uint32_t>() + FinishRoom::kBase;
    fa.cur = fin.as<uint32_t>() + FinishRoom::kCur;
    fa.when = fin.as<uint32_t>() + FinishRoom::kWhen;
    fa.pos = fin.as<uint32_t>() + FinishRoom::kPos;
    fa.val = reinterpret_cast<uint16_t *>(fin.as<uint32_t>() + FinishRoom::kVal);
    fa.falls = fin.as<uint32_t>() + FinishRoom::kFalls;
    fa.level = level;
    fa.queue = queue;
    fa.bar = lbar + kBarWords;
    fa.ctl = ctl;
    // as many blocks as the most vertices it can get fill (co-resident: one per CU)
    const unsigned fgrid = std::min<unsigned>(std::min<unsigned>((unsigned)ctx->num_cus, FinishRoom::kBlocks),
                                              grid_for(std::min(n, tail_cap), kPerWave * (kBlock / 64)));
    void *fargs[] = {&fa};
    DT_HIP(hipLaunchCooperativeKernel((const void *)k_peel_finish, dim3(fgrid), dim3(kBlock), fargs, 0, st));
    prof_end(ctx, kProfPeelTail, st);
    DT_TRY(ranks());
    if (h.left && !h.error) {   // it left them: level by level, the last ones in one workgroup
        const PeelStart from{(uint32_t)h.lres, h.ho_k, h.ho_tail, h.ho_rounds};
        static_assert(FinishRoom::kCells >= 2 * kLevelTail, "level boundaries fit the cells' room");
        if (from.left > kLevelTail) DT_TRY(grid_levels(from, kLevelTail));
        k_peel_levels<<<1, kBlock, 0, st>>>(rl, lb, lc, fa.base, level, queue, ctl);
        prof_end(ctx, kProfPeelTail, st);
        DT_HIP(hipGetLastError());
        DT_TRY(ranks());
    }
    if (h.error & 1u) return fail(DT_EDEVICE, "core peel barrier timed out");
    if (h.error) return fail(DT_EDEVICE, "core peel failed its consistency checks (code %u)", h.error);
    if (h.qtail != n) return fail(DT_EDEVICE, "core peel queued %u of %u vertices", h.qtail, n);
    g->kappa = h.kappa;
    g->peel_rounds = h.rounds;
    g->alg_bytes_peel = 16ull * n + 16ull * g->m_s;
    return DT_OK;
}

}  // namespace dt
