// K4, h >= 4: the clique tail, the rest of a peel once few vertices are alive.
//
// Most rounds of an h >= 4 peel are tiny (R-MAT scale 18, h = 4: 12,400
// rounds, the median one removes one vertex with about a hundred alive
// neighbours, 99 % of them with at most 65,536 vertices alive), so a round
// costs its chain of launches and its longest serial loop, not its work.
// Here the alive vertices of every graph are renumbered (rank order kept)
// and their adjacency becomes a bit matrix, row v = v's neighbours.  With it
//   * the candidate set C_v of a removed vertex v is one row masked by the
//     live vertices: no list to scan, no stamps;
//   * an arc inside C_v is one bit test, |C_v|^2 of them, coalesced, instead
//     of a walk of every member's whole out-list with a search per entry;
//   * one workgroup per graph takes round after round (k_ct_engine), with
//     the live set, the frontier and a list of the lowest-degree vertices in
//     LDS, and no launch in between.
// A round too large for one workgroup is handed to every CU: the engine lists
// its vertices and stops, k_ct_edges writes the adjacency of every C_v as
// compact bitmap rows, k_ct_count counts and takes the losses off the
// degrees, and the next engine launch ends the round.  The host enqueues
// these three launches again and again without reading anything back but
// the number of unfinished graphs now and then.
//
// Owner rule, levels and rounds are those of the round kernels: a round
// removes every alive vertex of degree <= k; a clique with several of them is
// destroyed once, by the one of smallest rank; when none is left, k rises to
// the smallest alive degree (every round in the min-degree mode).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "engine.hpp"
#include "peel.hpp"

namespace dsd {

namespace {

constexpr int64_t CT_MAX = 131072;             // alive vertices per graph (2,048-word rows: live sets of 16 KB in LDS)
constexpr int64_t CT_SMALL = 16384;            // up to here a graph of a batch takes a 256-thread workgroup
constexpr int64_t CT_MATRIX_WORDS = (int64_t)1 << 29;   // all matrices together (4 GiB)
constexpr int64_t CT_ARENA_WORDS = (int64_t)1 << 25;    // compact rows of one handed-over round (256 MiB), at least
                                                        // one vertex's worth
constexpr int64_t CT_SHRINK_MIN = 4096;        // a matrix at least this wide is rebuilt once half its vertices are gone
constexpr int64_t CT_VERTICES = (int64_t)1 << 23;       // vertices of all graphs together (items fit the counter)
constexpr int CT_ITEM_SHIFT = 40;              // item counter above, task counter below in one 64-bit word
constexpr u64 CT_TASK_MASK = (1ull << CT_ITEM_SHIFT) - 1ull;
// One workgroup keeps a round whose vertices beyond 64 neighbours hold at
// most this many member pairs (sum of |C_v|^2); the grid's two launches and
// the engine's restart cost about 20 us, what one CU needs for 2^17 pairs.
constexpr u64 CT_LIGHT_PAIRS = 1ull << 17;

enum : int32_t { CT_ROUND = 0, CT_HEAVY = 1, CT_DONE = 2, CT_STOPPED = 3 };

// one graph: where its arrays lie, and its state between launches
struct CtGraph {
    int32_t g;            // graph index of the peel
    int32_t base;         // first local vertex (ldeg, glob, hlist)
    int32_t A, AW;        // vertices, 64-bit words per matrix row
    int64_t moff, boff;   // first word of the matrix, of the live and current sets
    u64 k, mu;
    int64_t n_alive, nF;  // nF: frontier of the round in progress
    int32_t nlevels, rounds, open, phase;
    int32_t nheavy;       // frontier vertices still to be handed to the grid (hlist[hsel])
    int32_t hsel;
    u64 dest;             // cliques destroyed in this round, counted once per member besides their owner
};

// a vertex handed to the grid: its members' local ids and compact rows in the arena
struct CtItem {
    int32_t gi, d, W, pad;
    u64 task0;            // first member task
    int64_t off;          // word offset: ceil(d / 2) words of member ids, then d rows of W words
};

struct CtCtl {
    u64 count[2];                  // items << CT_ITEM_SHIFT | member tasks, by parity
    unsigned long long atop[2];    // arena words handed out
    int32_t ndone;                 // graphs finished or stopped
    int32_t nstop;                 // stopped for a smaller matrix
    int32_t err;
    u64 pairs, hand, hpairs;       // member pairs tested in the engine; vertices and pairs handed over
};

struct CtBufs {
    CtCtl *ctl;
    CtGraph *cg;
    int32_t *glob;        // local -> vertex
    u64 *ldeg;            // clique-degrees
    u64 *M;               // matrices
    u64 *lb, *cb;         // live and current (frontier) sets between launches
    int32_t *hlist[2];
    CtItem *items[2];
    u64 *arena;
    int64_t acap;
    int32_t R;            // h - 1: a removed vertex destroys the R-cliques of its C_v
    int32_t minpeel;
    u64 light;
};

// words per compact row: at R >= 4 a width the counting is compiled for
__host__ __device__ __forceinline__ int ct_words(int R, int d) {
    const int w = (d + 63) >> 6;
    if (R == 3) return w;
    return w <= 2 ? 2 : w <= 4 ? 4 : w <= 8 ? 8 : w;
}

// ---------------------------------------------------------------- counting

// word w (uniform) of the set M, without an indexed access to its registers
template <int W>
__device__ __forceinline__ u64 ct_pick(const u64 (&M)[W], int w) {
    u64 v = M[0];
#pragma unroll
    for (int q = 1; q < W; q++) v = w == q ? M[q] : v;
    return v;
}

// cliques of size D inside the set M (rank order); the sets stay in
// registers (every index a constant), S: rows with stride ws
template <int D, int W>
__device__ __forceinline__ u64 ct_count_in(const u64 (&M)[W], const u64 *S, int ws) {
    if constexpr (D == 1) {
        u64 c = 0;
#pragma unroll
        for (int q = 0; q < W; q++) c += (u64)__popcll(M[q]);
        return c;
    } else {
        u64 tot = 0;
#pragma unroll 1
        for (int w = 0; w < W; w++) {
            u64 word = ct_pick<W>(M, w);
            while (word) {
                const int bit = __builtin_ctzll(word);
                word &= word - 1;
                const u64 *row = S + (size_t)(w * 64 + bit) * ws;
                u64 M2[W];
#pragma unroll
                for (int q = 0; q < W; q++) M2[q] = q < w ? 0ull : ((q == w ? word : M[q]) & row[q]);   // above the bit
                tot += ct_count_in<D - 1, W>(M2, S, ws);
            }
        }
        return tot;
    }
}

__device__ __forceinline__ u64 bcast64(u64 v, int src) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src);
    return ((u64)hi << 32) | lo;
}

// The R-cliques of the set {0 .. d-1} (rows S, stride ws, W words, symmetric)
// that hold member i, on one wave: the (R-1)-cliques among its neighbours.
// Lane j of each 64 takes neighbour y = 64 q + j.
template <int R, int W>
__device__ __forceinline__ u64 ct_member_small(int i, int d, const u64 *S, int ws) {
    const int L = lane();
    u64 N[W];
    const u64 mine = L < W ? S[(size_t)i * ws + L] : 0ull;
#pragma unroll
    for (int q = 0; q < W; q++) N[q] = bcast64(mine, q);
    u64 c = 0;
#pragma unroll 1
    for (int q = 0; q < W; q++) {
        const u64 nq = bcast64(mine, q);
        if ((nq >> L) & 1ull) {
            const u64 *row = S + (size_t)(q * 64 + L) * ws;
            u64 M2[W];
            if constexpr (R == 3) {
                // every pair of adjacent neighbours from both its ends
#pragma unroll
                for (int w = 0; w < W; w++) M2[w] = N[w] & row[w];
                c += ct_count_in<1, W>(M2, S, ws);
            } else {
                const u64 above = L == 63 ? 0ull : (~0ull << (L + 1));
#pragma unroll
                for (int w = 0; w < W; w++) M2[w] = w < q ? 0ull : (N[w] & row[w] & (w == q ? above : ~0ull));
                c += ct_count_in<R - 2, W>(M2, S, ws);
            }
        }
    }
    c = wave_sum(c);
    return R == 3 ? c / 2 : c;
}

// The set bits of the words M (word w in lane w of every lane group of Wp
// lanes, w < W <= 64), 64 at a time through the wave's queue q (2 * WAVE ids):
// fn(take) with q[0, take) filled.
template <class F>
__device__ __forceinline__ void ct_bits(u64 M, int W, int32_t *q, F fn) {
    const int L = lane();
    int qn = 0;
    for (int w = 0; w < W; w++) {
        const u64 m = bcast64(M, w);
        if (!m) continue;
        if ((m >> L) & 1ull) q[qn + __popcll(m & lanemask_lt())] = w * 64 + L;
        qn += __popcll(m);
        __builtin_amdgcn_wave_barrier();
        if (qn >= WAVE) {
            fn(WAVE);
            const int rest = qn - WAVE;
            int32_t keep = 0;
            if (L < rest) keep = q[WAVE + L];
            __builtin_amdgcn_wave_barrier();
            if (L < rest) q[L] = keep;
            qn = rest;
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (qn > 0) fn(qn);
    __builtin_amdgcn_wave_barrier();
}

// pairs (y, z) with y in the queue and z in M and S[y], summed over this
// lane's words: lanes lie in groups of Wp, a group takes a y and its lanes the
// words of its row (coalesced), eight rows in flight
__device__ __forceinline__ u64 ct_drain(const int32_t *q, int take, u64 M, const u64 *S, int W, int lw) {
    const int L = lane(), Wp = 1 << lw, grp = L >> lw, w = L & (Wp - 1), G = WAVE >> lw;
    u64 c = 0;
    for (int u0 = 0; u0 < take; u0 += 8 * G) {
        u64 v[8];
#pragma unroll
        for (int t = 0; t < 8; t++) {
            const int u = u0 + t * G + grp;
            v[t] = (u < take && w < W) ? S[(size_t)q[u] * W + w] : 0ull;
        }
#pragma unroll
        for (int t = 0; t < 8; t++) c += (u64)__popcll(v[t] & M);
    }
    return c;
}

// the bits of word w above id y
__device__ __forceinline__ u64 ct_above(int w, int y) {
    const int yw = y >> 6;                             // (-1 for y = -1: every bit)
    if (w < yw) return 0ull;
    if (w > yw) return ~0ull;
    return (y & 63) == 63 ? 0ull : (~0ull << ((y & 63) + 1));
}

// D-cliques inside M (word w in lane w of every group), D >= 2, twice
// (the last pair is counted from both its ends), summed over all lanes of
// the wave.  qs: D - 1 queues of 2 * WAVE ids.
template <int D>
__device__ u64 ct_wide(u64 M, const u64 *S, int W, int lw, int32_t *qs) {
    u64 c = 0;
    ct_bits(M, W, qs, [&](int take) {
        if constexpr (D == 2) {
            c += ct_drain(qs, take, M, S, W, lw);
        } else {
            const int w = lane() & ((1 << lw) - 1);
            for (int t = 0; t < take; t++) {
                const int y = qs[t];
                const u64 row = w < W ? S[(size_t)y * W + w] : 0ull;
                c += ct_wide<D - 1>(M & row & ct_above(w, y), S, W, lw, qs + 2 * WAVE);
            }
        }
    });
    return c;
}

// The same for rows of more than 64 words: M is the intersection of the rows
// p[0 .. n-1] above id lo, its words read where they are needed.
template <int D, int n>
__device__ u64 ct_huge(const u64 *const *p, int lo, const u64 *S, int W) {
    auto word = [&](int w) {
        u64 m = ct_above(w, lo);
#pragma unroll
        for (int t = 0; t < n; t++) m &= p[t][w];
        return m;
    };
    u64 c = 0;
    for (int w0 = 0; w0 < W; w0++) {
        u64 m = word(w0);
        while (m) {
            const int y = w0 * 64 + __builtin_ctzll(m);
            m &= m - 1;
            const u64 *row = S + (size_t)y * W;
            if constexpr (D == 2) {
                for (int w = lane(); w < W; w += WAVE) c += (u64)__popcll(word(w) & row[w]);
            } else {
                const u64 *p2[n + 1];
#pragma unroll
                for (int t = 0; t < n; t++) p2[t] = p[t];
                p2[n] = row;
                c += ct_huge<D - 1, n + 1>(p2, y, S, W);
            }
        }
    }
    return c;
}

// ---------------------------------------------------------------- the grid's part of a large round

__device__ __forceinline__ int ct_item_of(const CtItem *items, int n, u64 task) {
    int lo = 0, hi = n - 1;                        // the largest item with task0 <= task
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].task0 <= task) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// One wave per member x of a handed-over vertex: x's compact row, one bit test per member of the
// set against x's matrix row, 64 members a ballot, eight in flight.  Bound by
// the latency of the row's sectors (a row of 16,384 columns is 2 KB, and 64
// ascending members share its lines).
__global__ __launch_bounds__(BLOCK) void k_ct_edges(CtBufs q, int par) {
    const u64 cnt = q.ctl->count[par];
    const int nitems = (int)(cnt >> CT_ITEM_SHIFT);
    const u64 ntask = cnt & CT_TASK_MASK;
    const CtItem *items = q.items[par];
    const int wv = threadIdx.x / WAVE, L = lane();
    for (u64 t = (u64)blockIdx.x * WAVES_PER_BLOCK + wv; t < ntask; t += (u64)gridDim.x * WAVES_PER_BLOCK) {
        const CtItem it = items[ct_item_of(items, nitems, t)];
        const CtGraph &cg = q.cg[it.gi];
        const int i = (int)(t - it.task0), d = it.d, W = it.W;
        const int32_t *C = (const int32_t *)(q.arena + it.off);
        u64 *row = q.arena + it.off + (d + 1) / 2 + (int64_t)i * W;
        const uint32_t *Mx = (const uint32_t *)(q.M + cg.moff + (int64_t)C[i] * cg.AW);
        for (int w0 = 0; w0 < W; w0 += 8) {
            uint32_t v[8];
            int32_t cj[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int j = (w0 + u) * 64 + L;
                cj[u] = j < d ? C[j] : -1;
            }
#pragma unroll
            for (int u = 0; u < 8; u++) v[u] = cj[u] >= 0 ? Mx[cj[u] >> 5] : 0u;
            u64 mine = 0;
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const u64 bw = __ballot(cj[u] >= 0 && ((v[u] >> (cj[u] & 31)) & 1u));
                if (L == u) mine = bw;
            }
            if (L < 8 && w0 + L < W) row[w0 + L] = mine;
        }
    }
}

// One wave per member: the cliques of its vertex that hold it, taken off its degree.
template <int R>
__global__ __launch_bounds__(BLOCK) void k_ct_count(CtBufs q, int par) {
    __shared__ int32_t sQ[WAVES_PER_BLOCK][(R - 2) * 2 * WAVE];
    __shared__ u64 sT[WAVES_PER_BLOCK];
    __shared__ int32_t sG[WAVES_PER_BLOCK];
    u64 tally = 0;        // the wave's members' counts, of the graph it last served
    int32_t tg = 0;
    const u64 cnt = q.ctl->count[par];
    const int nitems = (int)(cnt >> CT_ITEM_SHIFT);
    const u64 ntask = cnt & CT_TASK_MASK;
    const CtItem *items = q.items[par];
    const int wv = threadIdx.x / WAVE, L = lane();
    for (u64 t = (u64)blockIdx.x * WAVES_PER_BLOCK + wv; t < ntask; t += (u64)gridDim.x * WAVES_PER_BLOCK) {
        const CtItem it = items[ct_item_of(items, nitems, t)];
        const CtGraph &cg = q.cg[it.gi];
        const int i = (int)(t - it.task0), d = it.d, W = it.W;
        const int32_t x = ((const int32_t *)(q.arena + it.off))[i];
        const u64 *S = q.arena + it.off + (d + 1) / 2;
        u64 c;
        if (W <= 2 && R > 3) c = ct_member_small<R, 2>(i, d, S, W);
        else if (W == 4 && R > 3) c = ct_member_small<R, 4>(i, d, S, W);
        else if (W == 8 && R > 3) c = ct_member_small<R, 8>(i, d, S, W);
        else if (W <= 64) {
            int lw = 0;
            while ((1 << lw) < W) lw++;
            const int w = L & ((1 << lw) - 1);
            const u64 M = w < W ? S[(size_t)i * W + w] : 0ull;
            c = wave_sum(ct_wide<R - 1>(M, S, W, lw, sQ[wv])) / 2;
        } else {
            const u64 *p[1] = {S + (size_t)i * W};
            c = wave_sum(ct_huge<R - 1, 1>(p, -1, S, W)) / 2;
        }
        if (L == 0 && c) atomic_sub_u64(&q.ldeg[cg.base + x], c);
        if (it.gi != tg) {
            if (L == 0 && tally) atomicAdd(&q.cg[tg].dest, tally);
            tg = it.gi;
            tally = 0;
        }
        tally += c;
    }
    // one atomic per workgroup where its waves served one graph
    if (L == 0) {
        sT[wv] = tally;
        sG[wv] = tg;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 0; i < WAVES_PER_BLOCK; i++) {
            u64 v = sT[i];
            for (int j = i + 1; j < WAVES_PER_BLOCK; j++)
                if (sG[j] == sG[i]) {
                    v += sT[j];
                    sT[j] = 0;
                }
            if (v) atomicAdd(&q.cg[sG[i]].dest, v);
        }
}

// ---------------------------------------------------------------- the engine

// a graph's degrees are touched by its own workgroup only while the engine
// runs: the subtraction needs no wider scope, the load must pass the L1
__device__ __forceinline__ u64 ct_load_deg(const u64 *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 ct_sub_deg(u64 *p, u64 c) {
    return __hip_atomic_fetch_add(p, (u64)0 - c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// a degree's bin: exact below 16, then eight bins per power of two (monotone)
constexpr int CT_BINS = 512;
__device__ __forceinline__ int ct_bin(u64 d) {
    if (d < 16) return (int)d;
    const int e = 63 - __builtin_clzll(d);
    return (e - 2) * 8 + (int)((d >> (e - 3)) & 7ull);
}
// the largest degree of a bin
__device__ __forceinline__ u64 ct_bin_top(int b) {
    if (b < 16) return (u64)b;
    const int e = b / 8 + 2;
    return ((u64)(9 + (b & 7)) << (e - 3)) - 1ull;     // (bin 503: the top wraps to 2^64 - 1)
}

// One workgroup per graph.  CC: capacity of the candidate list, which holds
// every alive vertex of degree <= T (T raised when it runs dry): a round reads
// its degrees only.  DC: members of a C_v whose compact rows fit the LDS.
// AMAX: vertices of a graph.  A round is three workgroup barriers and about
// four dependent trips to L2 when its frontier has at most 64 neighbours
// each (a wave per vertex), four more barriers per larger vertex.
template <int BT, int CC, int DC, int AMAX, int R>
__global__ __launch_bounds__(BT) void k_ct_engine(PeelBufs b, CtBufs q, const int32_t *glist, int par, int64_t shrink_at) {
    constexpr int NW = BT / WAVE, WMAX = AMAX / 64, CPT = CC / BT, DW = DC / 64, DS = DW | 1;
    __shared__ u64 sLive[WMAX], sCur[WMAX];
    __shared__ int32_t sCand[2][CC], sF[CC];
    __shared__ u64 sS[DC * DS];
    __shared__ int32_t sC[DC];
    __shared__ u64 sCnt[DC];
    __shared__ int32_t sWC[NW][64];
    __shared__ u64 sWS[NW][64];
    __shared__ u64 sMin[NW];
    __shared__ int32_t sWsum[NW];
    __shared__ int32_t sN[2];                      // candidates of either list
    __shared__ int32_t sNF[2], sNfl[2], sNH[2];    // frontier, frontier with cliques, vertices beyond one wave
    __shared__ u64 sDest[2], sPairs[2];
    __shared__ int32_t sMaxD[2], sTook;
    const int gi = glist ? glist[blockIdx.x] : (int)blockIdx.x;
    const int t = threadIdx.x, wv = t / WAVE, L = lane();
    if (blockIdx.x == 0 && t == 0) {
        // the other parity's hand-over has been consumed by the launches before this one
        q.ctl->count[par ^ 1] = 0;
        q.ctl->atop[par ^ 1] = 0;
    }
    CtGraph &cg = q.cg[gi];
    int32_t phase = cg.phase;
    if (phase >= CT_DONE) return;
    const int32_t A = cg.A, AW = cg.AW, base = cg.base;
    const u64 *M = q.M + cg.moff;
    u64 *ldeg = q.ldeg + base;
    u64 k = cg.k, mu = cg.mu;
    int64_t n_alive = cg.n_alive, nF = cg.nF;
    int32_t nlevels = cg.nlevels, rounds = cg.rounds, nheavy = cg.nheavy, hsel = cg.hsel;
    bool open = cg.open != 0;
    const int64_t lv_base = b.gs[cg.g].lv_base;
    for (int w = t; w < AW; w += BT) {
        sLive[w] = q.lb[cg.boff + w];
        sCur[w] = q.cb[cg.boff + w];
    }
    if (t < 2) {
        sN[t] = 0;
        sNF[t] = sNfl[t] = sNH[t] = sMaxD[t] = 0;
        sDest[t] = sPairs[t] = 0;
    }
    __syncthreads();
    u64 T = 0, work = 0;
    u64 dest = phase == CT_HEAVY ? __hip_atomic_load(&cg.dest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    bool rescan = true;
    int cb = 0, p = 0;
    int64_t guard = 0;

    // the members of v's candidate set in word w: live, not a frontier vertex of rank <= v
    auto cand_word = [&](int32_t v, int w) -> u64 {
        const u64 m = M[(int64_t)v * AW + w];
        const int vw = v >> 6;
        u64 own = sCur[w];
        if (w > vw) own = 0;
        else if (w == vw) own &= (v & 63) == 63 ? ~0ull : ((2ull << (v & 63)) - 1ull);
        return m & sLive[w] & ~own;
    };
    auto apply = [&](int32_t x, u64 c) {
        const u64 old = ct_sub_deg(&ldeg[x], c);
        if (old > T && old - c <= T) {
            const int pos = atomicAdd(&sN[cb ^ 1], 1);
            if (pos < CC) sCand[cb ^ 1][pos] = x;
        }
    };

    while (true) {
        if (++guard > 4 * (int64_t)A + 64) {        // every pass ends a round or hands vertices over
            if (t == 0) q.ctl->err = 1;
            phase = CT_DONE;
            break;
        }
        if (phase == CT_HEAVY) {
            if (nheavy > 0) {
                // hand the listed vertices to the grid: members and a place for
                // their rows; those that find no room wait for the next launch
                if (t == 0) sTook = 0;
                __syncthreads();
                const int32_t *in = q.hlist[hsel] + base;
                int32_t *left = q.hlist[hsel ^ 1] + base;
                for (int j = wv; j < nheavy; j += NW) {
                    const int32_t v = in[j];
                    int c = 0;
                    for (int w = L; w < AW; w += WAVE) c += __popcll(cand_word(v, w));
                    const int d = wave_sum(c);
                    if (d < R) continue;
                    const int W = ct_words(R, d);
                    const int64_t words = (d + 1) / 2 + (int64_t)d * W;
                    int64_t off = -1;
                    int idx = -1;
                    u64 tb = 0;
                    if (L == 0) {
                        off = (int64_t)atomicAdd(&q.ctl->atop[par], (unsigned long long)words);
                        if (off + words <= q.acap) {
                            const u64 old = atomicAdd(&q.ctl->count[par], (1ull << CT_ITEM_SHIFT) | (u64)d);
                            idx = (int)(old >> CT_ITEM_SHIFT);
                            tb = old & CT_TASK_MASK;
                            q.items[par][idx] = CtItem{gi, d, W, 0, tb, off};
                            work += (u64)d * (u64)d;
                        } else {
                            left[atomicAdd(&sTook, 1)] = v;
                        }
                    }
                    idx = __shfl(idx, 0, WAVE);
                    if (idx < 0) continue;
                    off = __shfl(off, 0, WAVE);
                    int32_t *C = (int32_t *)(q.arena + off);
                    int run = 0;
                    for (int w0 = 0; w0 < AW; w0 += WAVE) {
                        u64 m = w0 + L < AW ? cand_word(v, w0 + L) : 0ull;
                        const int pc = __popcll(m);
                        const int inc = wave_incl_scan(pc);
                        int o = run + inc - pc;
                        while (m) {
                            C[o++] = (w0 + L) * 64 + __builtin_ctzll(m);
                            m &= m - 1;
                        }
                        run += __shfl(inc, WAVE - 1, WAVE);
                    }
                }
                __syncthreads();
                nheavy = sTook;
                hsel ^= 1;
                if (L == 0 && work) atomicAdd(&q.ctl->hpairs, work);
                if (t == 0) atomicAdd(&q.ctl->hand, 1ull);
                break;                               // the grid takes them
            }
            // every vertex of the round has been counted: it ends
            phase = CT_ROUND;
            rescan = true;
        } else {
            if (n_alive == 0) {
                phase = CT_DONE;
                break;
            }
            if (n_alive <= shrink_at) {
                phase = CT_STOPPED;
                break;
            }
            // ---- the level: smallest candidate degree
            int32_t cid[CPT];
            u64 cd[CPT];
            u64 gmin = ~0ull;
            if (!rescan) {
                const int nc = min(sN[cb], CC);
                if (sN[cb] > CC) rescan = true;      // (uniform: every thread reads the same count)
#pragma unroll
                for (int j = 0; j < CPT; j++) {
                    const int i = j * BT + t;
                    cid[j] = i < nc ? sCand[cb][i] : -1;
                    cd[j] = cid[j] >= 0 ? ct_load_deg(&ldeg[cid[j]]) : ~0ull;
                    gmin = cd[j] < gmin ? cd[j] : gmin;
                }
                gmin = wave_min(gmin);
                if (L == 0) sMin[wv] = gmin;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < NW; j++) gmin = sMin[j] < gmin ? sMin[j] : gmin;
                if (gmin == ~0ull) rescan = true;    // the list ran dry
            }
            bool mass = false;
            if (rescan) {
                // a new threshold: the smallest degree, then the largest bin
                // edge below which about half a list of vertices lies
                __syncthreads();
                uint32_t *hist = (uint32_t *)sS;     // (not in use between rounds)
                for (int i = t; i < CT_BINS; i += BT) hist[i] = 0;
                u64 m = ~0ull;
                __syncthreads();
                for (int l = t; l < A; l += BT) {
                    if (!((sLive[l >> 6] >> (l & 63)) & 1ull)) continue;
                    const u64 d = ct_load_deg(&ldeg[l]);
                    m = d < m ? d : m;
                    atomicAdd(&hist[ct_bin(d)], 1u);
                }
                m = wave_min(m);
                if (L == 0) sMin[wv] = m;
                __syncthreads();
                gmin = sMin[0];
                for (int j = 1; j < NW; j++) gmin = sMin[j] < gmin ? sMin[j] : gmin;
                const u64 need = (!b.minpeel && k > gmin) ? k : gmin;
                // every wave alike: a lane sums CT_BINS / WAVE bins
                constexpr int BL = CT_BINS / WAVE;
                uint32_t hs = 0, hb[BL];
#pragma unroll
                for (int i = 0; i < BL; i++) hs += hb[i] = hist[L * BL + i];
                uint32_t acc = wave_incl_scan(hs) - hs;
                int bin = -1;
#pragma unroll
                for (int i = 0; i < BL; i++) {
                    acc += hb[i];
                    if (acc <= CC / 2) bin = L * BL + i;
                }
                bin = wave_max(bin);
                T = bin >= 0 ? ct_bin_top(bin) : 0;
                if (T < need) T = need;
                if (t == 0) {
                    sN[0] = 0;
                    sN[1] = 0;
                }
                cb = 0;
                __syncthreads();
                for (int l = t; l < A; l += BT) {
                    if (!((sLive[l >> 6] >> (l & 63)) & 1ull)) continue;
                    const u64 d = ct_load_deg(&ldeg[l]);
                    if (d > T) continue;
                    const int pos = atomicAdd(&sN[0], 1);
                    if (pos < CC) sCand[0][pos] = l;
                }
                __syncthreads();
                const int nc = sN[0];
                mass = nc > CC;
                rescan = mass;
                if (!mass) {
#pragma unroll
                    for (int j = 0; j < CPT; j++) {
                        const int i = j * BT + t;
                        cid[j] = i < nc ? sCand[0][i] : -1;
                        cd[j] = cid[j] >= 0 ? ct_load_deg(&ldeg[cid[j]]) : ~0ull;
                    }
                }
            }
            if (b.minpeel || gmin > k) {             // no vertex at the level: a new one opens
                open = true;
                k = (b.minpeel || gmin > k) ? gmin : k;
            }
            if (open && t == 0) {
                const int64_t at = lv_base + nlevels;
                b.lv_k[at] = k;
                b.lv_size[at] = (u64)n_alive;
                b.lv_mu[at] = mu;
            }
            const u64 label = b.minpeel ? (u64)rounds : k;
            p ^= 1;
            if (mass) {
                // more vertices at or below the level than a list holds: the
                // frontier is marked by a pass over all of them and handed over
                int32_t *hl = q.hlist[hsel] + base;
                for (int l = t; l < A; l += BT) {
                    if (!((sLive[l >> 6] >> (l & 63)) & 1ull)) continue;
                    const u64 d = ct_load_deg(&ldeg[l]);
                    if (d > k) continue;
                    atomicOr((unsigned long long *)&sCur[l >> 6], 1ull << (l & 63));
                    const int32_t v = q.glob[base + l];
                    b.core[v] = label;
                    b.stamp[v] = -1;
                    atomicAdd(&sNF[p], 1);
                    if (d) hl[atomicAdd(&sNH[p], 1)] = l;
                }
                __syncthreads();
                nF = sNF[p];
                nheavy = sNH[p];
                dest = 0;
                if (t == 0) {
                    sNF[p ^ 1] = sNfl[p ^ 1] = sNH[p ^ 1] = sMaxD[p ^ 1] = 0;
                    sDest[p ^ 1] = sPairs[p ^ 1] = 0;
                }
                phase = CT_HEAVY;
                __syncthreads();
                continue;
            }
            // ---- the frontier; the other candidates move to the next list
#pragma unroll
            for (int j = 0; j < CPT; j++) {
                const bool have = cid[j] >= 0, take = have && cd[j] <= k;
                const bool keep = have && !take, wk = take && cd[j] != 0;
                const u64 mk = __ballot(keep), mt = __ballot(take), mw = __ballot(wk);
                int bk = 0, bw = 0;
                if (L == 0) {
                    if (mk) bk = atomicAdd(&sN[cb ^ 1], __popcll(mk));
                    if (mt) atomicAdd(&sNF[p], __popcll(mt));
                    if (mw) bw = atomicAdd(&sNfl[p], __popcll(mw));
                }
                bk = __builtin_amdgcn_readfirstlane(bk);
                bw = __builtin_amdgcn_readfirstlane(bw);
                if (keep) sCand[cb ^ 1][bk + __popcll(mk & lanemask_lt())] = cid[j];
                if (wk) sF[bw + __popcll(mw & lanemask_lt())] = cid[j];
                if (take) {
                    const int32_t l = cid[j];
                    atomicOr((unsigned long long *)&sCur[l >> 6], 1ull << (l & 63));
                    const int32_t v = q.glob[base + l];
                    b.core[v] = label;
                    b.stamp[v] = -1;
                }
            }
            __syncthreads();
            nF = sNF[p];
            const int nf = sNfl[p];
            if (t == 0) {
                // the other parity's counters, read before this round's first barrier
                sNF[p ^ 1] = sNfl[p ^ 1] = sNH[p ^ 1] = sMaxD[p ^ 1] = 0;
                sDest[p ^ 1] = sPairs[p ^ 1] = 0;
            }
            // every alive vertex leaves: no survivor's degree can fall, nothing to count
            const int nfw = nF == n_alive ? 0 : nf;
            // ---- a wave per frontier vertex: count C_v, and at most 64 members at once
            for (int f = wv; f < nfw; f += NW) {
                const int32_t v = sF[f];
                int c = 0;
                for (int w = L; w < AW; w += WAVE) c += __popcll(cand_word(v, w));
                const int d = wave_sum(c);
                if (d < R) continue;
                if (d > 64) {
                    if (L == 0) {
                        q.hlist[hsel][base + atomicAdd(&sNH[p], 1)] = v;
                        atomicAdd(&sPairs[p], (u64)d * (u64)d);
                        atomicMax(&sMaxD[p], d);
                    }
                    continue;
                }
                int run = 0;
                for (int w0 = 0; w0 < AW; w0 += WAVE) {
                    u64 m = w0 + L < AW ? cand_word(v, w0 + L) : 0ull;
                    if (__ballot(m != 0) == 0) continue;
                    const int pc = __popcll(m);
                    const int inc = wave_incl_scan(pc);
                    int o = run + inc - pc;
                    while (m) {
                        sWC[wv][o++] = (w0 + L) * 64 + __builtin_ctzll(m);
                        m &= m - 1;
                    }
                    run += __shfl(inc, WAVE - 1, WAVE);
                }
                __builtin_amdgcn_wave_barrier();
                const int32_t x = L < d ? sWC[wv][L] : 0;
                const uint32_t *M32 = (const uint32_t *)M;
                u64 row = 0;
                for (int i0 = 0; i0 < d; i0 += 8) {
                    uint32_t vv[8];
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const int32_t xi = __builtin_amdgcn_readlane(x, (i0 + u) & 63);
                        vv[u] = (i0 + u < d && L < d) ? M32[(int64_t)xi * AW * 2 + (x >> 5)] : 0u;
                    }
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const u64 bw = __ballot(L < d && ((vv[u] >> (x & 31)) & 1u));
                        if (L == i0 + u) row = bw;
                    }
                }
                sWS[wv][L] = row;
                __builtin_amdgcn_wave_barrier();
                u64 cx = 0;
                if (L < d) {
                    const u64 m1[1] = {row};
                    cx = ct_count_in<R - 1, 1>(m1, sWS[wv], 1);
                }
                if (cx) apply(x, cx);
                const u64 tot = wave_sum(cx);
                if (L == 0) {
                    if (tot) atomicAdd(&sDest[p], tot);
                    work += (u64)d * (u64)d;
                }
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            dest = 0;
            const int nh = sNH[p];
            if (nh > 0) {
                if (sMaxD[p] > DC || sPairs[p] > q.light) {
                    nheavy = nh;
                    dest = sDest[p];
                    phase = CT_HEAVY;
                    continue;                        // (the barrier above ordered hlist)
                }
                // ---- larger C_v one after another, the whole workgroup on each
                for (int f = 0; f < nh; f++) {
                    const int32_t v = q.hlist[hsel][base + f];
                    const int per = (AW + BT - 1) / BT, w0 = min(AW, t * per), w1 = min(AW, w0 + per);
                    int c = 0;
                    for (int w = w0; w < w1; w++) c += __popcll(cand_word(v, w));
                    const int inc = wave_incl_scan(c);
                    if (L == WAVE - 1) sWsum[wv] = inc;
                    __syncthreads();
                    int o = inc - c, d = 0;
                    for (int j = 0; j < NW; j++) {
                        if (j < wv) o += sWsum[j];
                        d += sWsum[j];
                    }
                    for (int w = w0; w < w1; w++) {
                        u64 m = cand_word(v, w);
                        while (m) {
                            sC[o++] = w * 64 + __builtin_ctzll(m);
                            m &= m - 1;
                        }
                    }
                    __syncthreads();
                    const int W = (d + 63) >> 6;
                    const uint32_t *M32 = (const uint32_t *)M;
                    for (int i = wv; i < d; i += NW) {
                        const uint32_t *Mx = M32 + (int64_t)sC[i] * AW * 2;
                        uint32_t vv[DW];
                        int32_t cj[DW];
#pragma unroll
                        for (int u = 0; u < DW; u++) {
                            const int j = u * 64 + L;
                            cj[u] = j < d ? sC[j] : -1;
                            vv[u] = cj[u] >= 0 ? Mx[cj[u] >> 5] : 0u;
                        }
                        u64 mine = 0;
#pragma unroll
                        for (int u = 0; u < DW; u++) {
                            const u64 bw = __ballot(cj[u] >= 0 && ((vv[u] >> (cj[u] & 31)) & 1u));
                            if (L == u) mine = bw;
                        }
                        if (L < DW) sS[i * DS + L] = mine;
                    }
                    __syncthreads();
                    u64 mydest = 0;
                    for (int i = wv; i < d; i += NW) {
                        u64 cx;
                        if (W <= 2) cx = ct_member_small<R, 2>(i, d, sS, DS);
                        else if (W <= 4) cx = ct_member_small<R, 4>(i, d, sS, DS);
                        else cx = ct_member_small<R, (DW < 4 ? 4 : DW)>(i, d, sS, DS);
                        if (L == 0) {
                            sCnt[i] = cx;
                            mydest += cx;
                        }
                    }
                    if (L == 0) {
                        if (mydest) atomicAdd(&sDest[p], mydest);
                        if (wv == 0) work += (u64)d * (u64)d;
                    }
                    __syncthreads();
                    for (int i = t; i < d; i += BT) {
                        const u64 cx = sCnt[i];
                        if (cx) apply(sC[i], cx);
                    }
                }
                __syncthreads();
            }
            dest = sDest[p];
            cb ^= 1;
        }
        // ---- the end of the round
        if (nF == n_alive) mu = 0;
        else mu -= dest / (u64)R;
        n_alive -= nF;
        nlevels += open ? 1 : 0;
        rounds += 1;
        open = false;
        dest = 0;
        if (rescan) {
            // a round that marked or changed many: clear the frontier everywhere
            __syncthreads();
            for (int w = t; w < AW; w += BT) {
                sLive[w] &= ~sCur[w];
                sCur[w] = 0;
            }
            __syncthreads();
        } else {
            // few frontier vertices: each thread still holds its own (in the
            // words it marked); the words are cleared whole by their first owner
            for (int w = t; w < AW; w += BT) {
                const u64 m = sCur[w];
                if (m) {
                    sLive[w] &= ~m;
                    sCur[w] = 0;
                }
            }
            if (t == 0) sN[cb ^ 1] = 0;              // the list just consumed becomes the next round's target
        }
    }
    __syncthreads();
    // the state, for the next launch
    for (int w = t; w < AW; w += BT) {
        q.lb[cg.boff + w] = sLive[w];
        q.cb[cg.boff + w] = sCur[w];
    }
    if (phase == CT_STOPPED)
        for (int l = t; l < A; l += BT)
            if ((sLive[l >> 6] >> (l & 63)) & 1ull) b.deg[q.glob[base + l]] = ct_load_deg(&ldeg[l]);
    if (phase != CT_HEAVY && L == 0 && work) atomicAdd(&q.ctl->pairs, work);
    if (t == 0) {
        cg.k = k;
        cg.mu = mu;
        cg.n_alive = n_alive;
        cg.nF = nF;
        cg.nlevels = nlevels;
        cg.rounds = rounds;
        cg.open = open ? 1 : 0;
        cg.phase = phase;
        cg.nheavy = nheavy;
        cg.hsel = hsel;
        cg.dest = dest;
        if (phase >= CT_DONE) {
            GraphState &g = b.gs[cg.g];
            g.k = k;
            g.kcand = ~0ull;
            g.mu_alive = mu;
            g.destroyed = 0;
            g.destroyed_m = 0;
            g.n_alive = n_alive;
            g.nF[0] = g.nF[1] = 0;
            g.nlevels = nlevels;
            g.sel = 0;
            atomicMax(&b.ctl->round, rounds);
            if (phase == CT_STOPPED) atomicAdd(&q.ctl->nstop, 1);
            atomicAdd(&q.ctl->ndone, 1);
        }
    }
}

// ---------------------------------------------------------------- preparation

// membership: alive, or in the pending frontier of the next round
__global__ void k_ct_flags(const int32_t *stamp, int32_t n, const PeelCtl *c, uint32_t *flag) {
    const int32_t r = c->round;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        flag[v] = stamp[v] >= r ? 1u : 0u;
}

__global__ void k_ct_glob(const uint32_t *flag, const uint32_t *loc, const u64 *deg, int32_t n, int32_t total,
                          int32_t *glob, u64 *ldeg, int32_t *err) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        if (v == n - 1 && (int64_t)loc[v] + flag[v] != total) *err = 2;
        if (!flag[v] || loc[v] >= (uint32_t)total) continue;
        glob[loc[v]] = (int32_t)v;
        ldeg[loc[v]] = deg[v];
    }
}

// the matrix, one workgroup per row: the row's bits gathered in LDS, then
// written whole; and the sets at their start (every vertex live)
__global__ __launch_bounds__(BLOCK) void k_ct_rows(PeelBufs b, CtBufs q, int32_t ng, int32_t total,
                                                   const uint32_t *flag, const uint32_t *loc) {
    __shared__ u64 sRow[CT_MAX / 64];
    for (int32_t l = blockIdx.x; l < total; l += gridDim.x) {
        int lo = 0, hi = ng - 1;                       // the graph: the largest with base <= l
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (q.cg[mid].base <= l) lo = mid;
            else hi = mid - 1;
        }
        const CtGraph &cg = q.cg[lo];
        const int32_t base = cg.base, A = cg.A, AW = cg.AW, v = q.glob[l];
        for (int w = threadIdx.x; w < AW; w += BLOCK) sRow[w] = 0;
        __syncthreads();
        const int64_t e1 = b.row_ptr[v + 1];
        for (int64_t e0 = b.row_ptr[v]; e0 < e1; e0 += 4 * BLOCK) {
            int32_t x[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t e = e0 + u * BLOCK + threadIdx.x;
                x[u] = e < e1 ? b.col[e] : -1;
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (x[u] < 0 || !flag[x[u]]) continue;
                const uint32_t j = loc[x[u]] - (uint32_t)base;
                if (j < (uint32_t)A) atomicOr((unsigned long long *)&sRow[j >> 6], 1ull << (j & 63));
            }
        }
        __syncthreads();
        u64 *row = q.M + cg.moff + (int64_t)(l - base) * AW;
        for (int w = threadIdx.x; w < AW; w += BLOCK) row[w] = sRow[w];
        if (l == base)
            for (int w = threadIdx.x; w < AW; w += BLOCK) {
                const int rem = A - w * 64;
                q.lb[cg.boff + w] = rem >= 64 ? ~0ull : ((1ull << rem) - 1ull);
                q.cb[cg.boff + w] = 0;
            }
        __syncthreads();
    }
}

__global__ void k_ct_close(PeelCtl *c, int32_t left) {
    c->n_alive = left;
    c->nF[0] = c->nF[1] = 0;
    c->nsel[0] = c->nsel[1] = 0;
    c->pending = 0;
}

template <int R>
void ct_sequence(const PeelBufs &b, const CtBufs &q, const int32_t *small, int nsmall, const int32_t *large, int nlarge,
                 int par, int64_t shrink_at, hipStream_t s) {
    if (nsmall) k_ct_engine<256, 1024, 256, (int)CT_SMALL, R><<<nsmall, 256, 0, s>>>(b, q, small, par, 0);
    if (nlarge) k_ct_engine<1024, 2048, 512, (int)CT_MAX, R><<<nlarge, 1024, 0, s>>>(b, q, large, par, shrink_at);
    k_ct_edges<<<1024, BLOCK, 0, s>>>(q, par);
    k_ct_count<R><<<1024, BLOCK, 0, s>>>(q, par);
    DSD_HIP(hipGetLastError());
}

}  // namespace

bool clique_tail(const PeelBufs &b, int h, int64_t n_alive, hipStream_t s, Scratch &sc, KernelTimes *kt) {
    const char *env = std::getenv("DSD_TAIL_ENGINE");
    if (env && std::strcmp(env, "0") == 0) return false;
    const int R = h - 1;
    bool first = true;
    while (true) {
        if (n_alive < 1 || n_alive > CT_VERTICES || (b.G == 1 && n_alive > CT_MAX)) return false;
        std::vector<GraphState> gs(b.G);
        DSD_HIP(hipMemcpyAsync(gs.data(), b.gs, (size_t)b.G * sizeof(GraphState), hipMemcpyDeviceToHost, s));
        int32_t round = 0;
        DSD_HIP(hipMemcpyAsync(&round, &b.ctl->round, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        DSD_HIP(hipStreamSynchronize(s));
        std::vector<CtGraph> cg;
        std::vector<int32_t> small, large;
        int64_t total = 0, words = 0, sets = 0, widest = 0;
        for (int32_t g = 0; g < b.G; g++) {
            const GraphState &st = gs[g];
            if (st.n_alive <= 0) continue;
            if (st.n_alive > CT_MAX) return false;
            CtGraph c{};
            c.g = g;
            c.base = (int32_t)total;
            c.A = (int32_t)st.n_alive;
            c.AW = (c.A + 63) / 64;
            c.moff = words;
            c.boff = sets;
            c.k = st.k;
            c.mu = st.mu_alive;
            c.n_alive = st.n_alive;
            c.nlevels = st.nlevels;
            c.rounds = round;
            c.open = st.sel != 0 ? 1 : 0;
            total += c.A;
            words += (int64_t)c.A * c.AW;
            sets += c.AW;
            widest = std::max<int64_t>(widest, c.A);
            (b.G > 1 && c.A <= CT_SMALL ? small : large).push_back((int32_t)cg.size());
            cg.push_back(c);
        }
        if (total != n_alive || words > CT_MATRIX_WORDS) {
            if (total != n_alive) throw Error(-3, "clique tail: the graphs' alive counts disagree with their sum");
            return false;
        }
        // a removed vertex's members with their compact rows, at worst all of its graph
        const int64_t one = widest / 2 + 1 + widest * std::max<int64_t>(8, (widest + 63) / 64);
        const int64_t acap = std::max<int64_t>(one, std::min<int64_t>(CT_ARENA_WORDS, 16 * words + (1 << 16)));
        if (first) {
            size_t free_b = 0, total_b = 0;
            const size_t need = 8 * (size_t)(words + acap + 2 * sets) + 96 * (size_t)total;
            if (hipMemGetInfo(&free_b, &total_b) != hipSuccess || need > free_b / 4) return false;
        }
        first = false;
        CtBufs q{};
        q.R = R;
        q.minpeel = b.minpeel;
        // with many graphs the other CUs have work of their own
        q.light = cg.size() >= 32 ? ~0ull : CT_LIGHT_PAIRS;
        q.acap = acap;
        q.ctl = sc.get_n<CtCtl>(1);
        q.cg = sc.get_n<CtGraph>((int64_t)cg.size());
        q.glob = sc.get_n<int32_t>(total);
        q.ldeg = sc.get_n<u64>(total);
        q.M = sc.get_n<u64>(words);
        q.lb = sc.get_n<u64>(sets);
        q.cb = sc.get_n<u64>(sets);
        q.hlist[0] = sc.get_n<int32_t>(total);
        q.hlist[1] = sc.get_n<int32_t>(total);
        q.items[0] = sc.get_n<CtItem>(total);
        q.items[1] = sc.get_n<CtItem>(total);
        q.arena = sc.get_n<u64>(acap);
        uint32_t *flag = sc.get_n<uint32_t>(b.n), *loc = sc.get_n<uint32_t>(b.n);
        int32_t *lists = sc.get_n<int32_t>((int64_t)cg.size());
        small.insert(small.end(), large.begin(), large.end());     // both lists in one upload
        const int nlarge = (int)large.size(), nsmall = (int)small.size() - nlarge;
        fill_i32((int32_t *)q.ctl, 0, (int64_t)(sizeof(CtCtl) / sizeof(int32_t)), s);
        DSD_HIP(hipMemcpyAsync(q.cg, cg.data(), cg.size() * sizeof(CtGraph), hipMemcpyHostToDevice, s));
        DSD_HIP(hipMemcpyAsync(lists, small.data(), small.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
        k_ct_flags<<<grid_for(b.n, BLOCK, 4096), BLOCK, 0, s>>>(b.stamp, b.n, b.ctl, flag);
        scan_exclusive_u32(flag, loc, b.n, s, sc);
        k_ct_glob<<<grid_for(b.n, BLOCK, 4096), BLOCK, 0, s>>>(flag, loc, b.deg, b.n, (int32_t)total, q.glob, q.ldeg,
                                                               &q.ctl->err);
        k_ct_rows<<<grid_for(total, 1, 8192), BLOCK, 0, s>>>(b, q, (int32_t)cg.size(), (int32_t)total, flag, loc);
        DSD_HIP(hipGetLastError());
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (kt && kt->time_main) {
            DSD_HIP(hipEventCreate(&e0));
            DSD_HIP(hipEventCreate(&e1));
            DSD_HIP(hipEventRecord(e0, s));
        }
        const int64_t shrink_at = b.G == 1 && widest >= CT_SHRINK_MIN ? widest / 2 : 0;
        CtCtl hc{};
        // a sequence ends every graph's round that the grid was given, so
        // they number at most the rounds; a vertex without room waits for the
        // next, and one always finds room
        int64_t seq = 0;
        int par = 0, chunk = 1;
        const int64_t max_seq = 4 * total + 64;
        while (true) {
            for (int i = 0; i < chunk; i++, par ^= 1) {
                switch (R) {
                    case 3: ct_sequence<3>(b, q, lists, nsmall, lists + nsmall, nlarge, par, shrink_at, s); break;
                    case 4: ct_sequence<4>(b, q, lists, nsmall, lists + nsmall, nlarge, par, shrink_at, s); break;
                    case 5: ct_sequence<5>(b, q, lists, nsmall, lists + nsmall, nlarge, par, shrink_at, s); break;
                    default: throw Error(-1, "h outside [4, 6]");
                }
            }
            seq += chunk;
            DSD_HIP(hipMemcpyAsync(&hc, q.ctl, sizeof(CtCtl), hipMemcpyDeviceToHost, s));
            DSD_HIP(hipStreamSynchronize(s));
            if (hc.err) throw Error(-3, hc.err == 2 ? "clique tail: the alive vertices disagree with their count"
                                                     : "clique tail: a round removed no vertex");
            if (hc.ndone == (int32_t)cg.size()) break;
            if (seq > max_seq) throw Error(-3, "clique tail did not converge");
            if (chunk < 16) chunk *= 2;
        }
        if (kt) {
            if (e0) {
                DSD_HIP(hipEventRecord(e1, s));
                DSD_HIP(hipEventSynchronize(e1));
                float ms = 0;
                DSD_HIP(hipEventElapsedTime(&ms, e0, e1));
                kt->tail_ms += ms;
                (void)hipEventDestroy(e0);
                (void)hipEventDestroy(e1);
            }
            kt->tail_launches += (u64)seq;
            kt->tail_pairs += hc.pairs;
            kt->tail_vertices += (u64)total;
            kt->tail_grid_rounds += hc.hand;
            kt->tail_grid_pairs += hc.hpairs;
        }
        if (!hc.nstop) {
            k_ct_close<<<1, 1, 0, s>>>(b.ctl, 0);
            return true;
        }
        GraphState g0;
        DSD_HIP(hipMemcpyAsync(&g0, b.gs, sizeof(GraphState), hipMemcpyDeviceToHost, s));
        DSD_HIP(hipStreamSynchronize(s));
        n_alive = g0.n_alive;
    }
}

}  // namespace dsd
