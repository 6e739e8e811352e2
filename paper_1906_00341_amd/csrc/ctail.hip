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
// its vertices and stops, k_ct_front lists the members of every C_v,
// k_ct_edges writes its adjacency as compact bitmap rows, k_ct_count counts
// and takes the losses off the degrees, and the next engine launch ends the
// round.  The host enqueues these four launches (five for a batch of small and
// large graphs, which take an engine of their own size) again and again
// without reading anything back but the number of unfinished graphs now and
// then.
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

constexpr int64_t CT_SMALL = 4096;             // up to here a graph of a batch takes the workgroup with smaller tables
constexpr int64_t CT_MID = 32768;              // up to here its waves buffer whole matrix rows in LDS
constexpr int64_t CT_ARENA_WORDS = (int64_t)1 << 25;    // compact rows of one handed-over round (256 MiB), at least
                                                        // one vertex's worth
constexpr int64_t CT_SHRINK_MIN = 4096;        // a matrix at least this wide is rebuilt once half its vertices are gone
constexpr int CT_ITEM_SHIFT = 40;              // item counter above, task counter below in one 64-bit word
constexpr u64 CT_TASK_MASK = (1ull << CT_ITEM_SHIFT) - 1ull;
// One workgroup keeps a round of at most CT_FRONT frontier vertices whose
// cost it puts at no more than CT_LIGHT: per vertex of d members, d matrix
// rows of AW words (a cycle each) and d^2 member pairs (a quarter of a cycle
// each; R > 3: d^3 / 64 for the counting; R = 5: d^4 / 64, as every triangle
// walks its common neighbours).  The grid's three launches and the engine's
// restart cost about as much (40 us).  h = 6 without the last term: rounds of
// milliseconds on one workgroup, core peel of R-MAT scale 16 / 17 2.67 / 9.84 s
// instead of 0.88 / 3.98 (CoreApp of scale 14 0.51 s instead of 0.15; none of
// the tail: 3.97 / 8.26 and 0.29); d^4 / 128 and / 256 measure 0.87 and 0.90 s
// at scale 16, 0.091 and 0.111 at scale 13 (d^4 / 64: 0.085).
constexpr u64 CT_LIGHT = (u64)CT_ROUND_CYCLES;
static_assert(CT_LIGHT >= 1000, "a price in cycles (not a phase)");
constexpr int CT_FRONT = 32;
// Two waves per SIMD: what every wave does alike (the level, the frontier,
// the control between barriers) is issued by each of them, so sixteen waves
// take it twice as long; one wave per SIMD leaves the latency of its own
// instructions open.  core of R-MAT scale 18, h = 4 / scale 16, h = 5: 256
// threads 361 / 264 ms, 512 303 / 193 ms; 1,024 (an earlier form) 394 / 303.
constexpr int CT_BLOCK = 512;
constexpr int CT_VS = 64;                      // vertices of one LDS batch

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
    int32_t nheavy;       // frontier vertices the grid found no room for (hlist[hsel])
    int32_t hsel;
    u64 dest;             // cliques destroyed in this round, counted once per member besides their owner
    u64 T;                // the candidate list across a hand-over: its threshold and vertices (cand);
    int32_t ncand, pad;   // -1: none kept
};

// a vertex handed to the grid, and (CtItem) its members' local ids and compact rows in the arena
struct CtFront {
    int32_t gi, v;
};
struct CtItem {
    int32_t gi, d, W, pad;
    u64 task0;            // first member task
    int64_t off;          // word offset: ceil(d / 2) words of member ids, then d rows of W words
};

struct CtCtl {
    u64 count[2];                  // items << CT_ITEM_SHIFT | member tasks, by parity
    int32_t nfront[2];             // vertices handed over
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
    int32_t *cand;        // [vertices] candidate lists across hand-overs
    CtItem *items[2];
    CtFront *front[2];
    u64 *arena;
    int64_t acap;
    int32_t R;            // h - 1: a removed vertex destroys the R-cliques of its C_v
    int32_t minpeel;
};

// words per compact row: at R >= 4 a width the counting is compiled for
__host__ __device__ __forceinline__ int ct_words(int R, int d) {
    const int w = (d + 63) >> 6;
    if (R == 3) return w;
    return w <= 2 ? 2 : w <= 4 ? 4 : w;
}

// ---------------------------------------------------------------- counting

// cliques of size D inside the set M (rank order), the loops over words
// unrolled: an indexed access would move the sets out of registers; S: rows
// with stride st
template <int D, int W>
__device__ __forceinline__ u64 ct_count_in(const u64 (&M)[W], const u64 *S, int st) {
    u64 c = 0;
    if constexpr (D == 1) {
#pragma unroll
        for (int q = 0; q < W; q++) c += (u64)__popcll(M[q]);
    } else {
#pragma unroll
        for (int w = 0; w < W; w++) {
            u64 word = M[w];
            while (word) {
                const int bit = __builtin_ctzll(word);
                word &= word - 1;
                const u64 *row = S + (w * 64 + bit) * st;
                u64 M2[W];
#pragma unroll
                for (int q = 0; q < W; q++) M2[q] = q < w ? 0ull : ((q == w ? word : M[q]) & row[q]);   // above the bit
                c += ct_count_in<D - 1, W>(M2, S, st);
            }
        }
    }
    return c;
}

__device__ __forceinline__ u64 bcast64(u64 v, int src) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src);
    return ((u64)hi << 32) | lo;
}

// The R-cliques (R >= 4) of the set with rows S (stride st, W words,
// symmetric) that hold member i, on one wave: the (R-1)-cliques among its
// neighbours.  Lane j of each 64 takes neighbour y = 64 q + j.
template <int R, int W>
__device__ __forceinline__ u64 ct_member_small(int i, const u64 *S, int st) {
    const int L = lane();
    u64 N[W];
    const u64 mine = L < W ? S[(size_t)i * st + L] : 0ull;
#pragma unroll
    for (int q = 0; q < W; q++) N[q] = bcast64(mine, q);
    u64 c = 0;
#pragma unroll 1
    for (int q = 0; q < W; q++) {
        const u64 nq = bcast64(mine, q);
        if ((nq >> L) & 1ull) {
            const u64 *row = S + (size_t)(q * 64 + L) * st;
            const u64 above = L == 63 ? 0ull : (~0ull << (L + 1));
            u64 M2[W];
#pragma unroll
            for (int w = 0; w < W; w++) M2[w] = w < q ? 0ull : (N[w] & row[w] & (w == q ? above : ~0ull));
            c += ct_count_in<R - 2, W>(M2, S, st);
        }
    }
    return wave_sum(c);
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
    u64 pairs = 0;
    for (u64 t = (u64)blockIdx.x * WAVES_PER_BLOCK + wv; t < ntask; t += (u64)gridDim.x * WAVES_PER_BLOCK) {
        const CtItem it = items[ct_item_of(items, nitems, t)];
        const CtGraph &cg = q.cg[it.gi];
        const int i = (int)(t - it.task0), d = it.d, W = it.W;
        pairs += (u64)d;
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
    if (L == 0 && pairs) atomicAdd(&q.ctl->hpairs, pairs);
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
        CtGraph &cg = q.cg[it.gi];
        const bool keep = cg.ncand >= 0;              // (only grows while >= 0)
        const int i = (int)(t - it.task0), d = it.d, W = it.W;
        const int32_t x = ((const int32_t *)(q.arena + it.off))[i];
        const u64 *S = q.arena + it.off + (d + 1) / 2;
        u64 c;
        if (R > 3 && W <= 2) c = ct_member_small<R, 2>(i, S, W);
        else if (R > 3 && W <= 4) c = ct_member_small<R, 4>(i, S, W);
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
        // (a removed vertex's degree slot holds its label)
        if (L == 0 && c && !((q.cb[cg.boff + (x >> 6)] >> (x & 63)) & 1ull)) {
            const u64 old = atomic_sub_u64(&q.ldeg[cg.base + x], c);
            // a vertex that crosses the threshold becomes a candidate (once: degrees only fall)
            if (keep && old > cg.T && old - c <= cg.T) q.cand[cg.base + atomicAdd(&cg.ncand, 1)] = x;
        }
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

// the members of v's candidate set in word w of its matrix row m: live, not a frontier vertex of rank <= v
__device__ __forceinline__ u64 ct_cand(u64 m, u64 live, u64 cur, int32_t v, int w) {
    const int vw = v >> 6;
    if (w > vw) cur = 0;
    else if (w == vw) cur &= (v & 63) == 63 ? ~0ull : ((2ull << (v & 63)) - 1ull);
    return m & live & ~cur;
}

// One wave per handed-over vertex: its members' ids to the arena, and an
// item with one task per member; a vertex without room goes back to its
// graph's list for the next sequence (the first one always finds room).
__global__ __launch_bounds__(BLOCK) void k_ct_front(CtBufs q, int par) {
    const int nf = q.ctl->nfront[par], L = lane();
    for (int f = blockIdx.x * WAVES_PER_BLOCK + threadIdx.x / WAVE; f < nf; f += gridDim.x * WAVES_PER_BLOCK) {
        const CtFront fr = q.front[par][f];
        CtGraph &cg = q.cg[fr.gi];
        const int32_t v = fr.v, AW = cg.AW;
        const u64 *row = q.M + cg.moff + (int64_t)v * AW, *lb = q.lb + cg.boff, *cb = q.cb + cg.boff;
        int c = 0;
        for (int w = L; w < AW; w += WAVE) c += __popcll(ct_cand(row[w], lb[w], cb[w], v, w));
        const int d = wave_sum(c);
        if (d < q.R) continue;
        const int W = ct_words(q.R, d);
        const int64_t words = (d + 1) / 2 + (int64_t)d * W;
        int64_t off = -1;
        if (L == 0) {
            off = (int64_t)atomicAdd(&q.ctl->atop[par], (unsigned long long)words);
            if (off + words <= q.acap) {
                const u64 old = atomicAdd(&q.ctl->count[par], (1ull << CT_ITEM_SHIFT) | (u64)d);
                q.items[par][old >> CT_ITEM_SHIFT] = CtItem{fr.gi, d, W, 0, old & CT_TASK_MASK, off};
            } else {
                off = -1;
                q.hlist[cg.hsel ^ 1][cg.base + atomicAdd(&cg.nheavy, 1)] = v;
            }
        }
        off = __shfl(off, 0, WAVE);
        if (off < 0) continue;
        int32_t *C = (int32_t *)(q.arena + off);
        int run = 0;
        for (int w0 = 0; w0 < AW; w0 += WAVE) {
            const int w = w0 + L;
            u64 m = w < AW ? ct_cand(row[w], lb[w], cb[w], v, w) : 0ull;
            const int pc = __popcll(m);
            const int inc = wave_incl_scan(pc);
            int o = run + inc - pc;
            while (m) {
                C[o++] = w * 64 + __builtin_ctzll(m);
                m &= m - 1;
            }
            run += __shfl(inc, WAVE - 1, WAVE);
        }
    }
}

// ---------------------------------------------------------------- the engine

// Wave reductions in VALU cross-lane operations (DPP): quad permutations and
// row mirrors reduce every 16-lane row, row broadcasts join the rows, lane 63
// ends with the total.
template <int CTRL, int MASK>
__device__ __forceinline__ int ct_dpp(int id, int v) {
    return __builtin_amdgcn_update_dpp(id, v, CTRL, MASK, 0xf, false);
}
__device__ __forceinline__ int ct_wave_sum(int v) {
    v += ct_dpp<0xb1, 0xf>(0, v);
    v += ct_dpp<0x4e, 0xf>(0, v);
    v += ct_dpp<0x141, 0xf>(0, v);
    v += ct_dpp<0x140, 0xf>(0, v);
    v += ct_dpp<0x142, 0xa>(0, v);
    v += ct_dpp<0x143, 0xc>(0, v);
    return __builtin_amdgcn_readlane(v, 63);
}
template <int CTRL, int MASK>
__device__ __forceinline__ u64 ct_min_step(u64 v) {
    const uint32_t lo = (uint32_t)ct_dpp<CTRL, MASK>(-1, (int)(uint32_t)v);
    const uint32_t hi = (uint32_t)ct_dpp<CTRL, MASK>(-1, (int)(uint32_t)(v >> 32));
    const u64 o = ((u64)hi << 32) | lo;
    return o < v ? o : v;
}
__device__ __forceinline__ u64 ct_wave_min(u64 v) {
    v = ct_min_step<0xb1, 0xf>(v);
    v = ct_min_step<0x4e, 0xf>(v);
    v = ct_min_step<0x141, 0xf>(v);
    v = ct_min_step<0x140, 0xf>(v);
    v = ct_min_step<0x142, 0xa>(v);
    v = ct_min_step<0x143, 0xc>(v);
    return bcast64(v, 63);
}
// exclusive prefix of a count 0 .. 64 over the wave's lanes, one ballot per bit
__device__ __forceinline__ int ct_wave_prefix(int v) {
    int pre = 0;
    const u64 lt = lanemask_lt();
#pragma unroll
    for (int bit = 0; bit < 7; bit++) pre += __popcll(__ballot((v >> bit) & 1) & lt) << bit;
    return pre;
}

// workgroup barrier that orders LDS only: global stores (core numbers) stay
// in flight across it; the degrees' atomics have returned by then
__device__ __forceinline__ void ct_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// a graph's degrees are touched by its own workgroup only while the engine runs
__device__ __forceinline__ u64 ct_load_deg(const u64 *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
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
    return ((u64)(9 + (b & 7)) << (e - 3)) - 1ull;     // (bin 495, the last one a degree has, and 511: 2^64 - 1)
}

// The edges (x, y), x < y, of the queue's codes (x << 16 | y, members of one
// vertex: rows at S, stride st), a lane each, R >= 4: every triangle (x, y, z),
// z above y, gives its corners the (R-3)-cliques of their common neighbours,
// so a member ends with C(R-1, 2) times its cliques.  (By edges alone a row
// would be read once for every z on either side: three times as many reads.)
template <int R, int W>
__device__ __forceinline__ void ct_edge_drain(const uint32_t *qu, int take, const u64 *S, int st, u64 *cnt) {
    const int L = lane();
    if (L < take) {
        const uint32_t code = qu[L];
        const int x = (int)(code >> 16), y = (int)(code & 0xffffu);
        u64 M[W], sum = 0;
#pragma unroll
        for (int w = 0; w < W; w++) M[w] = S[x * st + w] & S[y * st + w];
#pragma unroll
        for (int w = 0; w < W; w++) {
            u64 word = M[w] & ct_above(w, y);
            while (word) {
                // ZB corners at once: their rows are in flight together
                constexpr int ZB = W <= 2 ? 4 : 2;
                int z[ZB];
                u64 row[ZB][W];
#pragma unroll
                for (int u = 0; u < ZB; u++) {
                    z[u] = word ? w * 64 + __builtin_ctzll(word) : -1;
                    word &= word - 1;
                }
#pragma unroll
                for (int u = 0; u < ZB; u++)
#pragma unroll
                    for (int q = 0; q < W; q++) row[u][q] = S[max(z[u], 0) * st + q];
#pragma unroll
                for (int u = 0; u < ZB; u++) {
                    if (u > 0 && z[u] < 0) break;
                    u64 M2[W];
#pragma unroll
                    for (int q = 0; q < W; q++) M2[q] = M[q] & row[u][q];
                    const u64 c = ct_count_in<R - 3, W>(M2, S, st);
                    if (c) {
                        atomicAdd(&cnt[z[u]], c);
                        sum += c;
                    }
                }
            }
        }
        if (sum) {
            atomicAdd(&cnt[x], sum);
            atomicAdd(&cnt[y], sum);
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// R = 3: twice the triangles of the set that hold members i0 .. i0 + MB - 1, on
// one wave: for every neighbour y (a lane each) the neighbours it shares with
// the member.  y's row is read once for all MB members.
template <int W, int MB>
__device__ __forceinline__ void ct_member_tri(int i0, int n, int d, const u64 *S, int st, u64 *cnt) {
    const int L = lane();
    const u64 mine = S[(i0 + min(L / W, n - 1)) * st + L % W];
    u64 N[MB][W];
    uint32_t c[MB];
#pragma unroll
    for (int m = 0; m < MB; m++) {
        c[m] = 0;
#pragma unroll
        for (int q = 0; q < W; q++) N[m][q] = bcast64(mine, m * W + q);
    }
#pragma unroll
    for (int q = 0; q < W; q++) {
        u64 row[W];
        const u64 *y = S + min(q * 64 + L, d - 1) * st;
#pragma unroll
        for (int w = 0; w < W; w++) row[w] = y[w];
#pragma unroll
        for (int m = 0; m < MB; m++) {
            uint32_t s = 0;
#pragma unroll
            for (int w = 0; w < W; w++) s += (uint32_t)__popcll(N[m][w] & row[w]);
            c[m] += (N[m][q] >> L) & 1ull ? s : 0u;
        }
    }
    int tot = 0;
#pragma unroll
    for (int m = 0; m < MB; m++) {
        const int s = ct_wave_sum((int)c[m]);
        tot = L == m ? s : tot;
    }
    if (L < n) cnt[i0 + L] = (u64)(uint32_t)tot;
}

// words of a member's compact row in LDS, and their stride: odd beyond one
// word, so that the lanes' rows spread over the banks
__device__ __forceinline__ int ct_lds_words(int d) {
    const int W = (d + 63) >> 6;
    return W <= 2 ? W : W <= 4 ? 4 : 8;
}
__device__ __forceinline__ int ct_lds_stride(int Wt) { return Wt > 1 ? Wt + 1 : 1; }

// one batch of frontier vertices in LDS
struct CtBatch {
    u64 *S;               // the members' compact rows
    const int32_t *id;    // members, one vertex's after another
    const int32_t *vm, *vd, *vr;   // a vertex's first member, members, first row word
};

// The members' compact rows.  The words of a member's matrix row that hold
// members' columns (wlo on: the local ids follow the degree order, and the
// members of a low vertex are mostly hubs) are read coalesced, NWR a lane,
// laid into the wave's LDS buffer, and the members' bits gathered there:
// gathering from memory costs the CU about 36 cycles per 64 members whatever
// the row's width.  RB rows of one vertex go through together, the next RB
// are in flight meanwhile; the waves take such groups in turn.  While the
// matrix exceeds the XCD's L2 the one CU's misses bound this (about 8 bytes a
// cycle); then its instructions do.  Indexes are clamped rather than loads
// predicated: a predicated load gets a branch and a wait of its own.
constexpr int ct_rows_together(int nwr) { return nwr <= 2 ? 8 : 16 / nwr; }
template <int NWR, int WMAXT, int NW>
__device__ __forceinline__ void ct_rows_vertex(const CtBatch &B, int vm, int vd, int vr, int c0, const u64 *M, int AW,
                                               int wlo, u64 *buf) {
    constexpr int RB = ct_rows_together(NWR), BW = NWR * WAVE;
    const int L = lane();
    const uint32_t *b32 = (const uint32_t *)buf;
    int col[NWR];
#pragma unroll
    for (int c = 0; c < NWR; c++) col[c] = min(wlo + c * WAVE + L, AW - 1);
    // this lane's columns: word offset in the buffer, bit, and the lanes that hold one
    int off[WMAXT], sh[WMAXT];
    u64 have[WMAXT];
    const int Wt = ct_lds_words(vd), st = ct_lds_stride(Wt);
#pragma unroll
    for (int w = 0; w < WMAXT; w++) {
        const int32_t id = B.id[vm + min(w * WAVE + L, vd - 1)];
        off[w] = (id >> 5) - 2 * wlo;
        sh[w] = id & 31;
        have[w] = __ballot(w * WAVE + L < vd);
    }
    u64 r[RB][NWR];
    auto fetch = [&](int s0) {
        int64_t x[RB];
#pragma unroll
        for (int u = 0; u < RB; u++) x[u] = B.id[vm + min(s0 + u, vd - 1)];
#pragma unroll
        for (int u = 0; u < RB; u++)
#pragma unroll
            for (int c = 0; c < NWR; c++) r[u][c] = M[x[u] * AW + col[c]];
    };
    fetch(c0 * RB);
    for (int s0 = c0 * RB; s0 < vd; s0 += NW * RB) {
#pragma unroll
        for (int u = 0; u < RB; u++)
#pragma unroll
            for (int c = 0; c < NWR; c++) buf[u * BW + c * WAVE + L] = r[u][c];
        __builtin_amdgcn_wave_barrier();
        if (s0 + NW * RB < vd) fetch(s0 + NW * RB);
        u64 mine[RB];
#pragma unroll
        for (int u = 0; u < RB; u++) mine[u] = 0;
#pragma unroll
        for (int w = 0; w < WMAXT; w++) {
            if (w >= Wt) break;
            uint32_t v[RB];
#pragma unroll
            for (int u = 0; u < RB; u++) v[u] = b32[u * BW * 2 + off[w]];
#pragma unroll
            for (int u = 0; u < RB; u++) {
                const u64 bw = __ballot((v[u] >> sh[w]) & 1u) & have[w];
                mine[u] = L == w ? bw : mine[u];
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < RB; u++)
            if (L < Wt && s0 + u < vd) B.S[vr + (s0 + u) * st + L] = mine[u];
    }
}
template <int NWR, int NW>
__device__ __forceinline__ int ct_rows_do(const CtBatch &B, int vm, int vd, int vr, int first, const u64 *M, int AW,
                                           int wlo, u64 *buf) {
    constexpr int RB = ct_rows_together(NWR);
    const int chunks = (vd + RB - 1) / RB;
    if (first < chunks) {
        if (vd <= 64) ct_rows_vertex<NWR, 1, NW>(B, vm, vd, vr, first, M, AW, wlo, buf);
        else if (vd <= 256) ct_rows_vertex<NWR, 4, NW>(B, vm, vd, vr, first, M, AW, wlo, buf);
        else ct_rows_vertex<NWR, 8, NW>(B, vm, vd, vr, first, M, AW, wlo, buf);
    }
    return chunks;
}
// every vertex of the batch; WB: words of the longest row (0: no buffer, straight from memory)
template <int WB, int NW>
__device__ __forceinline__ void ct_rows(const CtBatch &B, int nv, const u64 *M, int AW, u64 *buf) {
    const int wv = threadIdx.x / WAVE, L = lane();
    const int lm = B.vm[L], ld = B.vd[L], lr = B.vr[L];        // (CT_VS = 64: a lane per vertex)
    int turn = wv;                                             // groups until this wave's next
    for (int vi = 0; vi < nv; vi++) {
        const int vm = __builtin_amdgcn_readlane(lm, vi), vd = __builtin_amdgcn_readlane(ld, vi),
                  vr = __builtin_amdgcn_readlane(lr, vi);
        const int wlo = __builtin_amdgcn_readfirstlane(B.id[vm]) >> 6, span = AW - wlo;
        int chunks;
        if constexpr (WB == 0) {
            // straight from memory: rows too long for a buffer (few rounds: most go to the grid)
            const int Wt = ct_lds_words(vd), st = ct_lds_stride(Wt);
            chunks = vd;
            for (int i = turn; i < vd; i += NW) {
                const uint32_t *x = (const uint32_t *)(M + (int64_t)B.id[vm + i] * AW);
                u64 mine = 0;
                for (int w = 0; w < Wt; w++) {
                    const int32_t id = B.id[vm + min(w * WAVE + L, vd - 1)];
                    const u64 bw = __ballot(((x[id >> 5] >> (id & 31)) & 1u) && w * WAVE + L < vd);
                    mine = L == w ? bw : mine;
                }
                if (L < Wt) B.S[vr + i * st + L] = mine;
            }
        } else if (WB <= 64 || span <= 64) {
            chunks = ct_rows_do<1, NW>(B, vm, vd, vr, turn, M, AW, wlo, buf);
        } else if (span <= 128) {
            chunks = ct_rows_do<2, NW>(B, vm, vd, vr, turn, M, AW, wlo, buf);
        } else if (span <= 256) {
            chunks = ct_rows_do<4, NW>(B, vm, vd, vr, turn, M, AW, wlo, buf);
        } else {
            chunks = ct_rows_do<8, NW>(B, vm, vd, vr, turn, M, AW, wlo, buf);
        }
        turn = (turn - chunks) & (NW - 1);                     // (NW a power of two)
    }
}

// One workgroup per graph.  CC: capacity of the candidate list, which holds
// every alive vertex of degree <= T (T raised when it runs dry): a round reads
// its degrees only.  SLOTS, ROWW, DC: members and row words of one batch of
// frontier vertices in LDS, members of one vertex.  AMAX: vertices of a graph.
// A round is six workgroup barriers and four dependent trips to L2: the
// candidates' degrees, the frontier's matrix rows, the members' rows, the
// degrees' atomics.
// WB: words of a matrix row that fit a wave's buffer (0: rows are not buffered).
template <int CC, int SLOTS, int ROWW, int AMAX, int WB, int R>
__global__ __launch_bounds__(CT_BLOCK) void k_ct_engine(PeelBufs b, CtBufs q, const int32_t *glist, int par, int64_t shrink_at) {
    constexpr int BT = CT_BLOCK, NW = BT / WAVE, WMAX = AMAX / 64, CPT = CC / BT;
    constexpr int DC = (R > 3 || SLOTS < 1024) ? 256 : 512;   // (R > 3: four-word sets in registers)
    static_assert(DC <= SLOTS && DC * (DC / 64 + 1) <= ROWW, "one vertex of DC members fits a batch");
    static_assert(WB == 0 || WB == WMAX, "a buffer holds the longest row");
    __shared__ u64 sLive[WMAX], sCur[WMAX];
    __shared__ int32_t sCand[2][CC], sF[CC];
    __shared__ u64 sS[ROWW];                       // compact rows, stride W + 1 (W > 1): odd, so lanes' rows spread over the banks
    __shared__ int32_t sId[SLOTS];                 // the batch's members, its vertices' one after another
    __shared__ u64 sCnt[SLOTS];
    __shared__ int32_t sVm[CT_VS], sVd[CT_VS], sVr[CT_VS];
    __shared__ uint32_t sQ[NW][R > 3 ? 2 * WAVE : 1];
    __shared__ u64 sRow[NW][WB > 64 ? 1024 : WB > 0 ? 512 : 1];   // eight rows of 64 words, down to two of 512
    __shared__ u64 sMin[NW];
    __shared__ u64 sAlloc[2];                      // vertices << 48 | members << 24 | row words, by batch parity
    __shared__ int32_t sSlots[2], sNv[2], sNext, sPend[2];
    __shared__ int32_t sN[2];                      // candidates of either list
    __shared__ int32_t sNF[2], sNfl[2], sNH[2];    // frontier, frontier with cliques, vertices for the grid
    __shared__ u64 sDest[2], sPairs[2];
    __shared__ uint32_t sHist[CT_BINS];
    __shared__ int32_t sAt, sYield;
    const int gi = glist ? glist[blockIdx.x] : (int)blockIdx.x;
    const int t = threadIdx.x, wv = t / WAVE, L = lane();
    if (blockIdx.x == 0 && t == 0) {
        // the other parity's hand-over has been consumed by the launches before this one
        q.ctl->count[par ^ 1] = 0;
        q.ctl->atop[par ^ 1] = 0;
        q.ctl->nfront[par ^ 1] = 0;
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
        sNF[t] = sNfl[t] = sNH[t] = sPend[t] = sSlots[t] = sNv[t] = 0;
        sDest[t] = sPairs[t] = sAlloc[t] = 0;
    }
    if (phase == CT_HEAVY) hsel ^= 1;              // what the grid sent back
    __syncthreads();
    const CtBatch batch{sS, sId, sVm, sVd, sVr};
    u64 T = 0, work = 0;
    u64 dest = phase == CT_HEAVY ? cg.dest : 0;
    bool rescan = true;
    int cb = 0, p = 0, turn = 0;
    int32_t kept = phase == CT_HEAVY ? cg.ncand : -1;   // candidates kept across the hand-over
    if (kept > CC) kept = -1;
    if (kept >= 0) {
        T = cg.T;
        for (int i = t; i < kept; i += BT) sCand[0][i] = q.cand[base + i];
        if (t == 0) sN[0] = kept;
    }
    __syncthreads();
    int64_t guard = 0;
    bool fresh = false;                             // the round in progress left a candidate list

    while (true) {
        if (++guard > 4 * (int64_t)A + 64) {        // every pass ends a round or hands vertices over
            if (t == 0) q.ctl->err = 1;
            phase = CT_DONE;
            break;
        }
        if (phase == CT_HEAVY) {
            if (nheavy > 0) {
                // hand the listed vertices to the grid, and keep the candidates
                // (list cb ^ 1 holds the round's survivors and newcomers)
                if (!fresh) kept = -1;
                else kept = sN[cb ^ 1] <= CC ? sN[cb ^ 1] : -1;
                for (int i = t; i < kept; i += BT) q.cand[base + i] = sCand[cb ^ 1][i];
                if (t == 0) sAt = atomicAdd(&q.ctl->nfront[par], nheavy);
                __syncthreads();
                for (int j = t; j < nheavy; j += BT)
                    q.front[par][sAt + j] = CtFront{gi, q.hlist[hsel][base + j]};
                if (t == 0) atomicAdd(&q.ctl->hand, 1ull);
                break;
            }
            // every vertex of the round has been counted: it ends, with the
            // candidate list as the grid left it, if it was kept
            phase = CT_ROUND;
            rescan = kept < 0;
            kept = -1;
        } else {
            if (n_alive == 0) {
                phase = CT_DONE;
                break;
            }
            if (n_alive <= shrink_at) {
                phase = CT_STOPPED;
                break;
            }
            // with other graphs waiting for the grid, the long runs of light
            // rounds are cut so that those do not wait for them one by one
            if (b.G > 1 && (++turn & 15) == 0) {
                if (t == 0) sYield = __hip_atomic_load(&q.ctl->nfront[par], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0;
                __syncthreads();
                const bool yield = sYield != 0;
                __syncthreads();
                if (yield) break;
            }
            // ---- the level: smallest candidate degree
            int32_t cid[CPT];
            u64 cd[CPT];
            u64 gmin = ~0ull;
            int nj = 0;                              // candidates of a thread
            if (!rescan) {
                const int nc = min(sN[cb], CC);
                if (sN[cb] > CC) rescan = true;      // (uniform: every thread reads the same count)
                nj = (nc + BT - 1) / BT;
#pragma unroll
                for (int j = 0; j < CPT; j++) {
                    if (j >= nj) break;
                    const int i = j * BT + t;
                    cid[j] = sCand[cb][min(i, nc - 1)];
                    cd[j] = ct_load_deg(&ldeg[cid[j]]);
                    if (i >= nc) {
                        cid[j] = -1;
                        cd[j] = ~0ull;
                    }
                }
#pragma unroll
                for (int j = 0; j < CPT; j++) {
                    if (j >= nj) break;
                    gmin = cd[j] < gmin ? cd[j] : gmin;
                }
                gmin = ct_wave_min(gmin);
                if (L == 0) sMin[wv] = gmin;
                ct_sync();
                gmin = sMin[0];
#pragma unroll
                for (int j = 1; j < NW; j++) gmin = sMin[j] < gmin ? sMin[j] : gmin;
                if (gmin == ~0ull) rescan = true;    // the list ran dry
            }
            bool mass = false;
            if (rescan) {
                // a new threshold: the smallest degree, then the largest bin
                // edge below which about half a list of vertices lies
                __syncthreads();
                for (int i = t; i < CT_BINS; i += BT) sHist[i] = 0;
                u64 m = ~0ull;
                __syncthreads();
                for (int l0 = t; l0 < A; l0 += 8 * BT) {
                    u64 d[8];
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const int l = l0 + u * BT;
                        d[u] = l < A && ((sLive[l >> 6] >> (l & 63)) & 1ull) ? ct_load_deg(&ldeg[l]) : ~0ull;
                    }
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        if (d[u] == ~0ull) continue;   // (no degree: a count of 2^64 - 1 cliques is refused)
                        m = d[u] < m ? d[u] : m;
                        atomicAdd(&sHist[ct_bin(d[u])], 1u);
                    }
                }
                m = ct_wave_min(m);
                if (L == 0) sMin[wv] = m;
                __syncthreads();
                gmin = sMin[0];
#pragma unroll
                for (int j = 1; j < NW; j++) gmin = sMin[j] < gmin ? sMin[j] : gmin;
                const u64 need = (!b.minpeel && k > gmin) ? k : gmin;
                // every wave alike: a lane sums CT_BINS / WAVE bins
                constexpr int BL = CT_BINS / WAVE;
                uint32_t hs = 0, hb[BL];
#pragma unroll
                for (int i = 0; i < BL; i++) hs += hb[i] = sHist[L * BL + i];
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
                for (int l0 = t; l0 < A; l0 += 8 * BT) {
                    u64 d[8];
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const int l = l0 + u * BT;
                        d[u] = l < A && ((sLive[l >> 6] >> (l & 63)) & 1ull) ? ct_load_deg(&ldeg[l]) : ~0ull;
                    }
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        if (d[u] == ~0ull || d[u] > T) continue;
                        const int pos = atomicAdd(&sN[0], 1);
                        if (pos < CC) sCand[0][pos] = l0 + u * BT;
                    }
                }
                __syncthreads();
                const int nc = sN[0];
                mass = nc > CC;
                rescan = mass;
                if (!mass) {
                    nj = (nc + BT - 1) / BT;
#pragma unroll
                    for (int j = 0; j < CPT; j++) {
                        if (j >= nj) break;
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
                    ldeg[l] = label;                 // a removed vertex's slot: its core number (or round)
                    atomicAdd(&sNF[p], 1);
                    if (d) hl[atomicAdd(&sNH[p], 1)] = l;
                }
                __syncthreads();
                nF = sNF[p];
                nheavy = nF == n_alive ? 0 : sNH[p];   // (every alive vertex leaves: nothing to count)
                dest = 0;
                if (t == 0) {
                    sNF[p ^ 1] = sNfl[p ^ 1] = sNH[p ^ 1] = 0;
                    sDest[p ^ 1] = sPairs[p ^ 1] = 0;
                }
                phase = CT_HEAVY;
                fresh = false;
                __syncthreads();
                continue;
            }
            // ---- the frontier; the other candidates move to the next list
#pragma unroll
            for (int j = 0; j < CPT; j++) {
                if (j >= nj) break;
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
                    ldeg[l] = label;                 // a removed vertex's slot: its core number (or round)
                }
            }
            if (t == 0) sNext = 0;
            ct_sync();
            nF = sNF[p];
            // every alive vertex leaves: no survivor's degree can fall, nothing to count
            const int nf = nF == n_alive ? 0 : sNfl[p];
            if (t == 0) {
                // the other parity's counters, read before this round's first barrier
                sNF[p ^ 1] = sNfl[p ^ 1] = sNH[p ^ 1] = 0;
                sDest[p ^ 1] = sPairs[p ^ 1] = 0;
            }
            if (nf > CT_FRONT) {
                for (int j = t; j < nf; j += BT) q.hlist[hsel][base + j] = sF[j];
                nheavy = nf;
                dest = 0;
                phase = CT_HEAVY;
                fresh = true;
                __syncthreads();
                continue;
            }
            // ---- batches of frontier vertices: list the members, compact the
            // rows, count, take the losses off the degrees
            int32_t hold = -1;                       // this wave's vertex that found no room in the last batch
            for (int bp = 0; nf > 0; bp ^= 1) {
                // a wave per vertex
                while (true) {
                    int32_t v = hold;
                    if (v < 0) {
                        int f = 0;
                        if (L == 0) f = atomicAdd(&sNext, 1);
                        f = __builtin_amdgcn_readfirstlane(f);
                        if (f >= nf) break;
                        v = sF[f];
                    }
                    hold = -1;
                    constexpr int WR = 4;            // row words a lane keeps (rows of at most 256 words)
                    u64 wr[WR];
                    int c = 0;
#pragma unroll
                    for (int u = 0; u < WR; u++) wr[u] = M[(int64_t)v * AW + min(u * WAVE + L, AW - 1)];
#pragma unroll
                    for (int u = 0; u < WR; u++) {
                        const int w = min(u * WAVE + L, AW - 1);
                        wr[u] = ct_cand(wr[u], sLive[w], sCur[w], v, w);
                        if (u * WAVE + L >= AW) wr[u] = 0;
                        c += __popcll(wr[u]);
                    }
                    for (int w = WR * WAVE + L; w < AW; w += WAVE)
                        c += __popcll(ct_cand(M[(int64_t)v * AW + w], sLive[w], sCur[w], v, w));
                    const int d = ct_wave_sum(c);
                    if (d < R) continue;
                    int vi = 0, m0 = 0, r0 = 0;
                    const int st = ct_lds_stride(ct_lds_words(d));
                    if (L == 0) {
                        const u64 dd = (u64)d * (u64)d;
                        const u64 pairs = (u64)d * (u64)AW + dd / 4 + (R > 3 ? dd * (u64)d / 64 : 0) + (R > 4 ? dd * dd / 64 : 0);
                        if (d > DC || atomicAdd(&sPairs[p], pairs) + pairs > CT_LIGHT) {
                            q.hlist[hsel][base + atomicAdd(&sNH[p], 1)] = v;
                            vi = -2;                 // the grid takes it
                        } else {
                            const u64 old = atomicAdd(&sAlloc[bp], (1ull << 48) | ((u64)d << 24) | (u64)(d * st));
                            vi = (int)(old >> 48);
                            m0 = (int)(old >> 24) & 0xffffff;
                            r0 = (int)(old & 0xffffff);
                            if (vi >= CT_VS || m0 + d > SLOTS || r0 + d * st > ROWW) {
                                atomicAdd(&sPairs[p], (u64)0 - pairs);
                                vi = -1;             // the next batch
                            } else {
                                sVm[vi] = m0;
                                sVd[vi] = d;
                                sVr[vi] = r0;
                                atomicMax(&sSlots[bp], m0 + d);
                                atomicMax(&sNv[bp], vi + 1);
                                work += dd;
                            }
                        }
                    }
                    vi = __builtin_amdgcn_readfirstlane(vi);
                    m0 = __builtin_amdgcn_readfirstlane(m0);
                    if (vi == -2) continue;
                    if (vi == -1) {
                        hold = v;
                        if (L == 0) atomicAdd(&sPend[bp], 1);
                        break;
                    }
                    int run = m0;
#pragma unroll
                    for (int u = 0; u < WR; u++) {
                        if (u * WAVE >= AW) break;
                        const int pc = __popcll(wr[u]);
                        int o = run + ct_wave_prefix(pc);
                        u64 m = wr[u];
                        while (m) {
                            sId[o] = (u * WAVE + L) * 64 + __builtin_ctzll(m);
                            sCnt[o] = 0;
                            o++;
                            m &= m - 1;
                        }
                        run += ct_wave_sum(pc);
                    }
                    for (int w0 = WR * WAVE; w0 < AW; w0 += WAVE) {
                        const int w = w0 + L;
                        u64 m = w < AW ? ct_cand(M[(int64_t)v * AW + w], sLive[w], sCur[w], v, w) : 0ull;
                        const int pc = __popcll(m);
                        int o = run + ct_wave_prefix(pc);
                        while (m) {
                            sId[o] = w * 64 + __builtin_ctzll(m);
                            sCnt[o] = 0;
                            o++;
                            m &= m - 1;
                        }
                        run += ct_wave_sum(pc);
                    }
                }
                ct_sync();
                const int slots = sSlots[bp], nv = sNv[bp];
                const bool more = sPend[bp] > 0;
                if (t == 0) {                        // the next batch's counters
                    sAlloc[bp ^ 1] = 0;
                    sSlots[bp ^ 1] = 0;
                    sNv[bp ^ 1] = 0;
                    sPend[bp ^ 1] = 0;
                }
                ct_rows<WB, NW>(batch, nv, M, AW, sRow[wv]);
                ct_sync();
                // count
                {
                    const int lm = sVm[L], ld = sVd[L], lr = sVr[L];
                    int turn = wv;
                    for (int vi = 0; vi < nv; vi++) {
                        const int m0 = __builtin_amdgcn_readlane(lm, vi), d = __builtin_amdgcn_readlane(ld, vi);
                        const int Wt = ct_lds_words(d), st = ct_lds_stride(Wt);
                        const u64 *S = sS + __builtin_amdgcn_readlane(lr, vi);
                        u64 *cn = sCnt + m0;
                        if constexpr (R == 3) {
                            int units;
                            // beyond 64 members on the matrix cores (d = 256: popcounts 62,000 cycles
                            // on one CU, products 10,000)
                            if (d <= 64) {
                                constexpr int MB = 8;
                                units = (d + MB - 1) / MB;
                                for (int g = turn; g < units; g += NW)
                                    ct_member_tri<1, MB>(g * MB, min(MB, d - g * MB), d, S, st, cn);
                            } else {
                                units = (d + 31) / 32;
                                for (int g = turn; g < units; g += NW) {
                                    if (d <= 128) tri_block<4>(g, d, S, st, cn);
                                    else if (DC <= 256 || d <= 256) tri_block<8>(g, d, S, st, cn);
                                    else tri_block<(DC <= 256 ? 8 : 16)>(g, d, S, st, cn);
                                }
                            }
                            turn = (turn - units) & (NW - 1);
                        } else {
                            // the wave gathers the edges of its members in a queue, a lane takes an edge
                            int qn = 0;
                            uint32_t *qu = sQ[wv];
                            auto drain = [&](int take) {
                                if (Wt == 1) ct_edge_drain<R, 1>(qu, take, S, st, cn);
                                else if (Wt == 2) ct_edge_drain<R, 2>(qu, take, S, st, cn);
                                else ct_edge_drain<R, 4>(qu, take, S, st, cn);
                            };
                            for (int i = turn; i < d; i += NW) {
                                const u64 mine = S[i * st + (L < Wt ? L : 0)];
                                for (int w = i >> 6; w < Wt; w++) {
                                    const u64 m = bcast64(mine, w) & ct_above(w, i);
                                    if (!m) continue;
                                    if ((m >> L) & 1ull)
                                        qu[qn + __popcll(m & lanemask_lt())] =
                                            ((uint32_t)i << 16) | (uint32_t)(w * 64 + L);
                                    qn += __popcll(m);
                                    __builtin_amdgcn_wave_barrier();
                                    if (qn >= WAVE) {
                                        drain(WAVE);
                                        const int rest = qn - WAVE;
                                        uint32_t keep = 0;
                                        if (L < rest) keep = qu[WAVE + L];
                                        __builtin_amdgcn_wave_barrier();
                                        if (L < rest) qu[L] = keep;
                                        qn = rest;
                                        __builtin_amdgcn_wave_barrier();
                                    }
                                }
                            }
                            if (qn) drain(qn);
                            turn = (turn - d) & (NW - 1);
                        }
                    }
                }
                ct_sync();
                for (int sl = t; sl < slots; sl += BT) {
                    const u64 c = sCnt[sl] / (u64)(R == 3 ? 2 : (R - 1) * (R - 2) / 2);
                    if (!c) continue;
                    const int32_t x = sId[sl];
                    atomicAdd(&sDest[p], c);
                    if ((sCur[x >> 6] >> (x & 63)) & 1ull) continue;   // leaves in this round
                    const u64 old = ct_sub_deg(&ldeg[x], c);
                    if (old > T && old - c <= T) {
                        const int pos = atomicAdd(&sN[cb ^ 1], 1);
                        if (pos < CC) sCand[cb ^ 1][pos] = x;
                    }
                }
                ct_sync();
                if (!more) break;
            }
            if (t == 0) {                            // the next round's first batch
                sAlloc[0] = sAlloc[1] = 0;
                sSlots[0] = sSlots[1] = 0;
                sNv[0] = sNv[1] = 0;
                sPend[0] = sPend[1] = 0;
            }
            dest = sDest[p];
            if (sNH[p] > 0) {
                nheavy = sNH[p];
                phase = CT_HEAVY;
                fresh = true;
                __syncthreads();                     // orders hlist
                continue;
            }
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
        if (rescan) __syncthreads();
        for (int w = t; w < AW; w += BT) {
            const u64 m = sCur[w];
            if (m) {
                sLive[w] &= ~m;
                sCur[w] = 0;
            }
        }
        if (rescan) __syncthreads();
        else if (t == 0) sN[cb ^ 1] = 0;             // the list just consumed becomes the next round's target
    }
    __syncthreads();
    // the state, for the next launch
    for (int w = t; w < AW; w += BT) {
        q.lb[cg.boff + w] = sLive[w];
        q.cb[cg.boff + w] = sCur[w];
    }
    if (phase >= CT_DONE)
        for (int l = t; l < A; l += BT) {
            const int32_t v = q.glob[base + l];
            const u64 x = ct_load_deg(&ldeg[l]);
            if ((sLive[l >> 6] >> (l & 63)) & 1ull) {
                b.deg[v] = x;                        // (only when stopped)
            } else {
                b.core[v] = x;
                b.stamp[v] = -1;
            }
        }
    if (L == 0 && work) atomicAdd(&q.ctl->pairs, work);
    if (t == 0) {
        cg.k = k;
        cg.mu = mu;
        cg.n_alive = n_alive;
        cg.nF = nF;
        cg.nlevels = nlevels;
        cg.rounds = rounds;
        cg.open = open ? 1 : 0;
        cg.phase = phase;
        cg.nheavy = 0;                               // (the grid counts those it finds no room for)
        cg.hsel = hsel;
        cg.dest = dest;
        cg.T = T;
        cg.ncand = kept;
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

// A batch's small graphs beside its large ones: the two engine launches of a
// sequence touch different graphs, so the small ones' goes to a stream of its
// own between two events (one after the other, 115 us of each sequence's 600 for
// 330 graphs).  The stream has drained before it goes.
struct CtFork {
    hipStream_t s2 = nullptr;
    hipEvent_t go = nullptr, done = nullptr;
    void open() {
        DSD_HIP(hipStreamCreateWithFlags(&s2, hipStreamNonBlocking));
        DSD_HIP(hipEventCreateWithFlags(&go, hipEventDisableTiming));
        DSD_HIP(hipEventCreateWithFlags(&done, hipEventDisableTiming));
    }
    ~CtFork() {
        if (s2) (void)hipStreamSynchronize(s2);
        if (go) (void)hipEventDestroy(go);
        if (done) (void)hipEventDestroy(done);
        if (s2) (void)hipStreamDestroy(s2);
    }
};

template <int R>
void ct_sequence(const PeelBufs &b, const CtBufs &q, const int32_t *small, int nsmall, const int32_t *large, int nlarge,
                 int64_t widest,
                 int par, int64_t shrink_at, hipStream_t s, const CtFork &fork) {
    if (fork.s2) {
        DSD_HIP(hipEventRecord(fork.go, s));
        DSD_HIP(hipStreamWaitEvent(fork.s2, fork.go, 0));
    }
    if (nsmall)
        k_ct_engine<1024, 512, 2560, (int)CT_SMALL, (int)CT_SMALL / 64, R>
            <<<nsmall, CT_BLOCK, 0, fork.s2 ? fork.s2 : s>>>(b, q, small, par, 0);
    if (fork.s2) DSD_HIP(hipEventRecord(fork.done, fork.s2));
    if (nlarge && widest <= CT_MID)
        k_ct_engine<2048, 1024, 5120, (int)CT_MID, (int)CT_MID / 64, R><<<nlarge, CT_BLOCK, 0, s>>>(b, q, large, par,
                                                                                                 shrink_at);
    else if (nlarge)
        k_ct_engine<2048, 1024, 5120, (int)CT_MAX, 0, R><<<nlarge, CT_BLOCK, 0, s>>>(b, q, large, par, shrink_at);
    if (fork.s2) DSD_HIP(hipStreamWaitEvent(s, fork.done, 0));
    k_ct_front<<<512, BLOCK, 0, s>>>(q, par);
    k_ct_edges<<<1024, BLOCK, 0, s>>>(q, par);
    k_ct_count<R><<<1024, BLOCK, 0, s>>>(q, par);
    DSD_HIP(hipGetLastError());
}

}  // namespace

bool clique_tail(const PeelBufs &b, int h, int64_t n_alive, hipStream_t s, Scratch &sc, KernelTimes *kt) {
    const char *env = std::getenv("DSD_TAIL_ENGINE");
    if (env && std::strcmp(env, "0") == 0) return false;
    const int R = h - 1;
    // allocated for the first matrix; those built again for fewer vertices fit
    // in the same buffers (a peel that is under way asks for no more memory)
    CtBufs q{};
    uint32_t *flag = nullptr, *loc = nullptr;
    int32_t *lists = nullptr;
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
        if (!q.ctl) {
            // DSD_CT_ARENA_WORDS overrides the arena size (0: room for one vertex)
            const char *aw = std::getenv("DSD_CT_ARENA_WORDS");
            const int64_t acap = std::max<int64_t>(
                one, aw ? std::atoll(aw) : std::min<int64_t>(CT_ARENA_WORDS, 16 * words + (1 << 16)));
            size_t free_b = 0, total_b = 0;
            const size_t need = 8 * (size_t)(words + acap + 2 * sets) + 112 * (size_t)total;
            if (hipMemGetInfo(&free_b, &total_b) != hipSuccess || need > free_b / 4 || !sc.may_take(need))
                return false;
            q.R = R;
            q.minpeel = b.minpeel;
            q.acap = acap;
            try {
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
                q.cand = sc.get_n<int32_t>(total);
                q.front[0] = sc.get_n<CtFront>(total);
                q.front[1] = sc.get_n<CtFront>(total);
                q.arena = sc.get_n<u64>(acap);
                flag = sc.get_n<uint32_t>(b.n);
                loc = sc.get_n<uint32_t>(b.n);
                lists = sc.get_n<int32_t>((int64_t)cg.size());
                q.ctl = sc.get_n<CtCtl>(1);
            } catch (const Error &e) {
                // another stream's work took the memory meanwhile: the round kernels go on
                if (e.status != -2 || sc.external()) throw;
                (void)hipGetLastError();
                return false;
            }
        }
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
        CtFork fork;
        if (nsmall && nlarge) fork.open();
        // a sequence ends every graph's round that the grid was given, so
        // they number at most the rounds; a vertex without room waits for the
        // next, and one always finds room
        int64_t seq = 0;
        int par = 0, chunk = 1;
        const int64_t max_seq = 4 * total + 64;
        while (true) {
            for (int i = 0; i < chunk; i++, par ^= 1) {
                switch (R) {
                    case 3: ct_sequence<3>(b, q, lists, nsmall, lists + nsmall, nlarge, widest, par, shrink_at, s, fork); break;
                    case 4: ct_sequence<4>(b, q, lists, nsmall, lists + nsmall, nlarge, widest, par, shrink_at, s, fork); break;
                    case 5: ct_sequence<5>(b, q, lists, nsmall, lists + nsmall, nlarge, widest, par, shrink_at, s, fork); break;
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
