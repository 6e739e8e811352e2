// Clique-counting engine over candidate sets (device templates).
//
// A work item names a root vertex w of the degree-ordered DAG.  Its
// candidate set C is N+(w) filtered by the item's context (a vertex mask for
// clique-degrees; "inside N(v) and still alive" for the peel).  The engine
// counts the R-cliques of the sub-DAG induced on C and attributes to every
// member x of C the number of those cliques that contain x; the item's
// prefix (w, and v for the peel) receives the total.  With R = h - 1 this is
// the clique-degree of Definition 3 restricted to cliques whose lowest-rank
// member is w; with R = h - 2 and prefix {v, w} it is the set of cliques
// through a removed vertex v that Algorithm 3 must take away.
//
// R = 1: every member of C completes one clique.
// R = 2: edges inside C, found by probing each x's out-list against an LDS
//        hash of C (no bitmap).
// R >= 3: the sub-DAG is stored as a symmetric bitmap S over C (local index
//        = rank order, so "out" = higher index).  Members in prefix positions
//        get their counts from popcounts of intersected rows; the last member
//        y of a clique gets, in one pass, the number of (R-1)-cliques inside
//        its in-neighbourhood Col(y).  No work is done per clique.  (The row
//        engine, R = 3 and 4 up to 1,088 and 768 members: the matrix cores
//        and a walk over triangles instead.)
//
// Context interface (Ctx):
//   int32_t root(int64_t item)                 -- w
//   bool accept(int64_t item, int32_t x)        -- x in N+(w) kept in C?
//   void add(int32_t x, u64 c)                  -- member x of c cliques
//   void add_prefix(int64_t item, u64 total)    -- the item's prefix, total cliques
#pragma once

#include "common.hpp"

namespace dsd {

constexpr int HASH_EMPTY = -1;

// ---------------------------------------------------------------- bit helpers

template <int W>
__device__ __forceinline__ u64 row_above(const u64 *S, int x, int w) {
    // bits of row x strictly above x (out-neighbours in the sub-DAG)
    u64 v = S[(size_t)x * W + w];
    int xw = x >> 6;
    if (w < xw) return 0;
    if (w == xw) return (x & 63) == 63 ? 0ull : (v & (~0ull << ((x & 63) + 1)));
    return v;
}

template <int W>
__device__ __forceinline__ u64 row_below(const u64 *S, int x, int w) {
    // bits of row x strictly below x (in-neighbours in the sub-DAG)
    u64 v = S[(size_t)x * W + w];
    int xw = x >> 6;
    if (w > xw) return 0;
    if (w == xw) return v & ((1ull << (x & 63)) - 1ull);
    return v;
}

template <int W>
__device__ __forceinline__ u64 popc_w(const u64 (&M)[W]) {
    u64 c = 0;
#pragma unroll
    for (int w = 0; w < W; w++) c += (u64)__popcll(M[w]);
    return c;
}

// number of D-cliques inside the candidate mask M (rank order, each once)
template <int D, int W>
__device__ u64 count_in(const u64 (&M)[W], const u64 *S) {
    if constexpr (D == 1) {
        return popc_w<W>(M);
    } else {
        u64 tot = 0;
#pragma unroll 1
        for (int w = 0; w < W; w++) {
            u64 word = M[w];
            while (word) {
                int x = w * 64 + __builtin_ctzll(word);
                word &= word - 1;
                u64 M2[W];
                bool any = false;
#pragma unroll
                for (int q = 0; q < W; q++) {
                    M2[q] = M[q] & row_above<W>(S, x, q);
                    any |= M2[q] != 0;
                }
                if (any) tot += count_in<D - 1, W>(M2, S);
            }
        }
        return tot;
    }
}

// Prefix enumeration: choose D more members from M; at D == 0 the number of
// completions is popc(M).  Every chosen member gets the completions through
// it (cnt is an LDS array of u64 counters).  Returns the total.
template <int D, int W>
__device__ u64 forward(const u64 (&M)[W], const u64 *S, u64 *cnt) {
    if constexpr (D == 0) {
        return popc_w<W>(M);
    } else {
        u64 tot = 0;
#pragma unroll 1
        for (int w = 0; w < W; w++) {
            u64 word = M[w];
            while (word) {
                int x = w * 64 + __builtin_ctzll(word);
                word &= word - 1;
                u64 M2[W];
                bool any = false;
#pragma unroll
                for (int q = 0; q < W; q++) {
                    M2[q] = M[q] & row_above<W>(S, x, q);
                    any |= M2[q] != 0;
                }
                if (!any) continue;
                u64 c = forward<D - 1, W>(M2, S, cnt);
                if (c) {
                    atomicAdd(&cnt[x], c);
                    tot += c;
                }
            }
        }
        return tot;
    }
}

// Per-member R-clique counts for the sub-DAG over d nodes stored in S
// (symmetric rows of W words).  Work item for one thread: node x.  Adds to
// cnt[] (LDS), returns the number of cliques whose first member is x.
template <int R, int W>
__device__ u64 bitmap_node_work(int x, const u64 *S, u64 *cnt) {
    u64 M[W];
    // x as first member
#pragma unroll
    for (int q = 0; q < W; q++) M[q] = row_above<W>(S, x, q);
    u64 c = forward<R - 2, W>(M, S, cnt);
    u64 tot = c;
    // x as last member: (R-1)-cliques inside its in-neighbourhood
#pragma unroll
    for (int q = 0; q < W; q++) M[q] = row_below<W>(S, x, q);
    c += count_in<R - 1, W>(M, S);
    if (c) atomicAdd(&cnt[x], c);
    return tot;
}

// ---------------------------------------------------------------- counts over LDS bitmaps

// Row sums of A o A^2 on the matrix cores: for every member j of a candidate
// set (0/1 adjacency A, rows S of stride st words, symmetric, zero bits past
// member d - 1), twice the triangles that hold j.  A unit is a column block J
// of 32 members: C = A[I] A[J]^T by 32 x 32 x 32 products of bytes for every
// row block I, then every lane adds its column's entries where A holds a 1.
// A byte comes from a bit by one AND: operand A keeps bit s of every byte at
// its place (value 2^s, s = 0..3, the other half wave's bits 4..7 shifted
// down), operand B moves it to place 3 - s, so that every product is 8.  A is
// symmetric, so both operands read rows, and the order of the k index does not
// matter as long as both take the same.  Rows past the last member repeat it;
// their products meet zero bits only.  Exact: a sum is at most 8 (d - 1)^2,
// below 2^32 far beyond the 2,048 members of any caller.  Bound by the matrix
// cores (32 cycles a product, five vector operations beside it).
typedef int tri_i4 __attribute__((ext_vector_type(4)));
typedef int tri_i16 __attribute__((ext_vector_type(16)));
template <int TMAX, class Cnt>
__device__ __forceinline__ void tri_block(int J, int d, const u64 *S, int st, Cnt *cnt) {
    const int L = lane(), lo = L & 31, sh = (L >> 5) * 4;
    const int T = (d + 31) >> 5;
    const int j = J * 32 + lo, jr = min(j, d - 1) * st;
    tri_i4 bj[TMAX];
#pragma unroll
    for (int k = 0; k < TMAX; k += 2) {
        if (k < T) {
            const u64 w = S[jr + (k >> 1)];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const uint32_t x = (uint32_t)(w >> (32 * h)) >> sh;
#pragma unroll
                for (int s = 0; s < 4; s++) bj[k + h][s] = (int)(((x >> s) & 0x01010101u) << (3 - s));
            }
        }
    }
    uint32_t sum = 0;
    for (int I = 0; I < T; I++) {
        const int ir = min(I * 32 + lo, d - 1) * st;
        // register r of the product holds row 8 (r / 4) + 4 (lane / 32) + r % 4
        const uint32_t mask = (uint32_t)(S[jr + (I >> 1)] >> (32 * (I & 1))) >> sh;
        tri_i16 acc = {};
#pragma unroll
        for (int k = 0; k < TMAX; k += 2) {
            if (k < T) {
                const u64 w = S[ir + (k >> 1)];
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const uint32_t x = (uint32_t)(w >> (32 * h)) >> sh;
                    tri_i4 a;
#pragma unroll
                    for (int s = 0; s < 4; s++) a[s] = (int)(x & (0x01010101u << s));
                    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, bj[k + h], acc, 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 16; r++) sum += (uint32_t)acc[r] & (0u - ((mask >> (8 * (r / 4) + r % 4)) & 1u));
    }
    if (j < d && sum) atomicAdd(&cnt[j], (Cnt)(sum >> 3));
}

// R = 4: the edges (x, y), x < y, of the queue's codes (x << 16 | y), a lane
// each: every triangle (x, y, z), z above y, gives its corners the number of
// their common neighbours, so a member ends with three times its 4-cliques.
template <int W>
__device__ __forceinline__ void quad_drain(const uint32_t *qu, int take, const u64 *S, int st, u64 *cnt) {
    const int L = lane();
    if (L < take) {
        const uint32_t code = qu[L];
        const int x = (int)(code >> 16), y = (int)(code & 0xffffu);
        const u64 *rx = S + x * st, *ry = S + y * st;
        u64 M[W], sum = 0;
#pragma unroll
        for (int w = 0; w < W; w++) M[w] = rx[w] & ry[w];
        for (int w = y >> 6; w < W; w++) {
            u64 word = rx[w] & ry[w];                    // (from LDS: an index into M would leave the registers)
            if (w == (y >> 6)) word &= (y & 63) == 63 ? 0ull : (~0ull << ((y & 63) + 1));
            while (word) {
                const int z = w * 64 + __builtin_ctzll(word);
                word &= word - 1;
                const u64 *rz = S + z * st;
                uint32_t c = 0;
#pragma unroll
                for (int q = 0; q < W; q++) c += (uint32_t)__popcll(M[q] & rz[q]);
                if (c) {
                    atomicAdd(&cnt[z], (u64)c);
                    sum += c;
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

// ---------------------------------------------------------------- LDS hash

__device__ __forceinline__ void hash_insert(int32_t *keys, int32_t *vals, int bits, int32_t x, int32_t v) {
    uint32_t m = (1u << bits) - 1u, slot = hash_slot(x, bits);
    while (true) {
        int32_t prev = atomicCAS(&keys[slot], HASH_EMPTY, x);
        if (prev == HASH_EMPTY || prev == x) {
            vals[slot] = v;
            return;
        }
        slot = (slot + 1) & m;
    }
}

__device__ __forceinline__ int32_t hash_find(const int32_t *keys, const int32_t *vals, int bits, int32_t x) {
    uint32_t m = (1u << bits) - 1u, slot = hash_slot(x, bits);
    while (true) {
        int32_t k = keys[slot];
        if (k == x) return vals[slot];
        if (k == HASH_EMPTY) return -1;
        slot = (slot + 1) & m;
    }
}

// ---------------------------------------------------------------- block helpers

// In-place inclusive scan of a[0, n) (n <= BLOCK * per) in LDS; returns total.
__device__ __forceinline__ int32_t block_incl_scan_lds(int32_t *a, int n, int32_t *wtmp) {
    int per = (n + BLOCK - 1) / BLOCK;
    int lo = threadIdx.x * per, hi = min(n, lo + per);
    int32_t s = 0;
    for (int i = lo; i < hi; i++) s += a[i];
    int32_t inc = wave_incl_scan(s);
    int w = threadIdx.x / WAVE;
    if (lane() == WAVE - 1) wtmp[w] = inc;
    __syncthreads();
    int32_t off = inc - s;
    for (int i = 0; i < w; i++) off += wtmp[i];
    int32_t total = 0;
    for (int i = 0; i < WAVES_PER_BLOCK; i++) total += wtmp[i];
    for (int i = lo; i < hi; i++) {
        off += a[i];
        a[i] = off;
    }
    __syncthreads();
    return total;
}

// ---------------------------------------------------------------- item kernels

// Load the candidate set of an item into out[] in rank order (order-preserving
// block compaction).  Returns |C|.  d <= cap.
template <class Ctx>
__device__ int block_load_candidates(const Ctx &ctx, int64_t item, const int32_t *col, int64_t s0, int d,
                                     int32_t *out, int32_t *wtmp) {
    int per = (d + BLOCK - 1) / BLOCK;
    int lo = threadIdx.x * per, hi = min(d, lo + per);
    int32_t keep = 0;
    for (int i = lo; i < hi; i++) keep += ctx.accept(item, col[s0 + i]) ? 1 : 0;
    int32_t inc = wave_incl_scan(keep);
    int w = threadIdx.x / WAVE;
    if (lane() == WAVE - 1) wtmp[w] = inc;
    __syncthreads();
    int32_t off = inc - keep;
    for (int i = 0; i < w; i++) off += wtmp[i];
    int32_t total = 0;
    for (int i = 0; i < WAVES_PER_BLOCK; i++) total += wtmp[i];
    for (int i = lo; i < hi; i++) {
        int32_t x = col[s0 + i];
        if (ctx.accept(item, x)) out[off++] = x;
    }
    __syncthreads();
    return total;
}

// ---- wave engine: one wave per item, d <= 64 ---------------------------------
// R = 2 uses the hash; R >= 3 the one-word bitmap.
template <int R, class Ctx>
__global__ __launch_bounds__(BLOCK) void k_engine_wave(Ctx ctx, const int64_t *row_ptr, const int32_t *col,
                                                       const int64_t *dag_off, int64_t nitems,
                                                       const int32_t *nitems_dev) {
    if (nitems_dev) nitems = *nitems_dev;
    __shared__ int32_t sC[WAVES_PER_BLOCK][64];
    __shared__ int32_t sKey[WAVES_PER_BLOCK][128];
    __shared__ int32_t sVal[WAVES_PER_BLOCK][128];
    __shared__ int32_t sPre[WAVES_PER_BLOCK][64];
    __shared__ int64_t sSt[WAVES_PER_BLOCK][64];
    __shared__ u64 sCnt[WAVES_PER_BLOCK][64];
    __shared__ u64 sS[WAVES_PER_BLOCK][64];
    const int wv = threadIdx.x / WAVE, L = lane();
    for (int i = L; i < 128; i += WAVE) sKey[wv][i] = HASH_EMPTY;
    sCnt[wv][L] = 0;
    sS[wv][L] = 0;
    __builtin_amdgcn_wave_barrier();
    const int64_t stride = (int64_t)gridDim.x * WAVES_PER_BLOCK;
    for (int64_t it = (int64_t)blockIdx.x * WAVES_PER_BLOCK + wv; it < nitems; it += stride) {
        const int32_t w = ctx.root(it);
        const int64_t s0 = dag_off[w];
        const int d = (int)(row_ptr[w + 1] - s0);
        int32_t x = -1;
        bool keep = false;
        if (L < d) {
            x = col[s0 + L];
            keep = ctx.accept(it, x);
        }
        const u64 km = __ballot(keep);
        const int dd = __popcll(km);
        if (dd < R) continue;                                   // wave-uniform
        const int li = __popcll(km & lanemask_lt());            // rank order kept
        if (keep) {
            sC[wv][li] = x;
            hash_insert(sKey[wv], sVal[wv], 7, x, li);
        }
        __builtin_amdgcn_wave_barrier();
        u64 total = 0;
        if constexpr (R == 1) {
            if (keep) ctx.add(x, 1);
            total = (u64)dd;
        } else {
            // flattened (i, offset) pairs over the out-lists of C
            int32_t len = 0;
            int64_t st = 0;
            if (keep) {
                st = dag_off[x];
                len = (int32_t)(row_ptr[x + 1] - st);
            }
            int32_t inc = wave_incl_scan(keep ? len : 0);
            if (keep) {
                sPre[wv][li] = inc;
                sSt[wv][li] = st;
            }
            const int32_t tot_pairs = __shfl(inc, WAVE - 1, WAVE);
            __builtin_amdgcn_wave_barrier();
            u64 hits = 0;
            for (int32_t base = 0; base < tot_pairs; base += WAVE) {
                int32_t p = base + L;
                bool hit = false;
                int i = 0, j = -1;
                if (p < tot_pairs) {
                    i = upper_bound_i32(sPre[wv], dd, p);
                    int32_t off = p - (i ? sPre[wv][i - 1] : 0);
                    int32_t y = col[sSt[wv][i] + off];
                    j = hash_find(sKey[wv], sVal[wv], 7, y);
                    hit = j >= 0;
                }
                if constexpr (R == 2) {
                    if (hit) {
                        atomicAdd(&sCnt[wv][i], 1ull);
                        atomicAdd(&sCnt[wv][j], 1ull);
                    }
                    hits += (u64)__popcll(__ballot(hit));
                } else {
                    if (hit) {
                        atomicOr(&sS[wv][i], 1ull << j);
                        atomicOr(&sS[wv][j], 1ull << i);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
            if constexpr (R == 2) {
                total = hits;
            } else {
                u64 t = 0;
                if (L < dd) t = bitmap_node_work<R, 1>(L, &sS[wv][0], &sCnt[wv][0]);
                total = wave_sum(t);
            }
            __builtin_amdgcn_wave_barrier();
            if (L < dd) {
                u64 c = sCnt[wv][L];
                if (c) ctx.add(sC[wv][L], c);
            }
        }
        if (L == 0 && total) ctx.add_prefix(it, total);
        __builtin_amdgcn_wave_barrier();
        // reset the wave's LDS for the next item
        for (int i = L; i < 128; i += WAVE) sKey[wv][i] = HASH_EMPTY;
        sCnt[wv][L] = 0;
        sS[wv][L] = 0;
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- block engine: one block per item -------------------------------------
// CAP: max |N+(w)|; HB: hash bits (2^HB >= 2*CAP); W: bitmap words (R >= 3);
// GLOBAL_S: the bitmap lives in a per-block slice of global scratch.
template <int R, int CAP, int HB, int W, bool GLOBAL_S, class Ctx>
__global__ __launch_bounds__(BLOCK) void k_engine_block(Ctx ctx, const int64_t *row_ptr, const int32_t *col,
                                                        const int64_t *dag_off, int64_t nitems,
                                                        const int32_t *nitems_dev, u64 *gS) {
    if (nitems_dev) nitems = *nitems_dev;
    __shared__ int32_t sC[CAP];
    __shared__ int32_t sKey[1 << HB];
    __shared__ int32_t sVal[1 << HB];
    __shared__ int32_t sPre[CAP];
    __shared__ u64 sCnt[CAP];
    __shared__ int32_t wtmp[WAVES_PER_BLOCK];
    __shared__ u64 sTot[WAVES_PER_BLOCK];
    constexpr int SW = (R >= 3 && !GLOBAL_S) ? CAP * W : 1;
    __shared__ u64 sSl[SW];
    u64 *S = GLOBAL_S ? gS + (size_t)blockIdx.x * CAP * W : sSl;
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const int32_t w = ctx.root(it);
        const int64_t s0 = dag_off[w];
        const int d = (int)(row_ptr[w + 1] - s0);
        for (int i = threadIdx.x; i < (1 << HB); i += BLOCK) sKey[i] = HASH_EMPTY;
        const int dd = block_load_candidates(ctx, it, col, s0, d, sC, wtmp);
        if (dd < R) continue;                                  // block-uniform
        for (int i = threadIdx.x; i < dd; i += BLOCK) {
            hash_insert(sKey, sVal, HB, sC[i], i);
            sCnt[i] = 0;
            int32_t x = sC[i];
            sPre[i] = (int32_t)(row_ptr[x + 1] - dag_off[x]);
        }
        if constexpr (R >= 3) {
            for (int i = threadIdx.x; i < dd * W; i += BLOCK) S[i] = 0;
        }
        __syncthreads();
        u64 total = 0;
        if constexpr (R == 1) {
            for (int i = threadIdx.x; i < dd; i += BLOCK) ctx.add(sC[i], 1);
            total = (u64)dd;
        } else {
            const int32_t tot_pairs = block_incl_scan_lds(sPre, dd, wtmp);
            u64 hits = 0;
            for (int32_t base = 0; base < tot_pairs; base += BLOCK) {
                int32_t p = base + threadIdx.x;
                if (p < tot_pairs) {
                    int i = upper_bound_i32(sPre, dd, p);
                    int32_t off = p - (i ? sPre[i - 1] : 0);
                    int32_t x = sC[i];
                    int32_t y = col[dag_off[x] + off];
                    int j = hash_find(sKey, sVal, HB, y);
                    if (j >= 0) {
                        if constexpr (R == 2) {
                            atomicAdd(&sCnt[i], 1ull);
                            atomicAdd(&sCnt[j], 1ull);
                            hits++;
                        } else {
                            atomicOr(&S[(size_t)i * W + (j >> 6)], 1ull << (j & 63));
                            atomicOr(&S[(size_t)j * W + (i >> 6)], 1ull << (i & 63));
                        }
                    }
                }
            }
            if constexpr (R >= 3) {
                if (GLOBAL_S) __threadfence_block();
                __syncthreads();
                for (int x = threadIdx.x; x < dd; x += BLOCK) hits += bitmap_node_work<R, W>(x, S, sCnt);
            }
            hits = wave_sum(hits);
            if (lane() == 0) sTot[threadIdx.x / WAVE] = hits;
            __syncthreads();
            for (int i = 0; i < WAVES_PER_BLOCK; i++) total += sTot[i];
            for (int i = threadIdx.x; i < dd; i += BLOCK) {
                u64 c = sCnt[i];
                if (c) ctx.add(sC[i], c);
            }
        }
        if (threadIdx.x == 0 && total) ctx.add_prefix(it, total);
        __syncthreads();
    }
}

// ---- row engine: one workgroup per item, a wave per member's out-list -------
// R = 2, 3, 4; CAP: max |N+(w)|; SB: 2^SB hash slots; W: bitmap words a row
// (R >= 3).  A wave walks N+(x) of one member x at a time, coalesced, four
// entries a lane in flight, and probes the hash of C: no search for the
// (member, entry) pair a lane holds, which took ten dependent LDS reads a
// pair.  A slot holds 20 bits of the entry's hash beside its index, so most
// misses end with one read.  R = 3 counts on the matrix cores (tri_block),
// R = 4 by triangles (quad_drain), R = 2 by the hits themselves.  Clique-
// degrees of R-MAT scale 22, h = 4 (2.9e10 probes): 400 -> 96 ms; of R-MAT
// scale 18, h = 5: 139 -> 17 ms, against a search per pair, one thread per
// member and 64-bit LDS atomics per prefix.
template <int R, int CAP, int SB, int W, int BT, class Ctx>
__global__ __launch_bounds__(BT) void k_engine_rows(Ctx ctx, const int64_t *row_ptr, const int32_t *col,
                                                    const int64_t *dag_off, int64_t nitems) {
    constexpr int NW = BT / WAVE, ST = W | 1;
    __shared__ u64 sS[R >= 3 ? CAP * ST : 1];
    __shared__ int32_t sC[CAP];
    __shared__ uint32_t sH[1 << SB];
    __shared__ u64 sCnt64[R >= 4 ? CAP : 1];
    __shared__ uint32_t sQ[NW][R >= 4 ? 2 * WAVE : 1];
    __shared__ int32_t sWsum[NW];
    __shared__ u64 sTot[NW];
    static_assert((1 << SB) >= CAP && CAP <= 2048, "indexes fit a slot, counters the table");
    uint32_t *cnt = sH;                                // R = 3: the table's space, once it has been used
    __shared__ uint32_t sCnt2[R == 2 ? CAP : 1];       // (a member's edges: at most CAP - 1)
    const int t = threadIdx.x, wv = t / WAVE, L = lane();
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const int32_t w = ctx.root(it);
        const int64_t s0 = dag_off[w];
        const int d = (int)(row_ptr[w + 1] - s0);
        for (int i = t; i < (1 << SB); i += BT) sH[i] = 0;
        // candidates, rank order kept
        int dd = 0;
        for (int i0 = 0; i0 < d; i0 += BT) {
            const int i = i0 + t;
            const int32_t x = i < d ? col[s0 + i] : -1;
            const bool ok = i < d && ctx.accept(it, x);
            const u64 m = __ballot(ok);
            if (L == 0) sWsum[wv] = __popcll(m);
            __syncthreads();
            int at = dd + __popcll(m & lanemask_lt());
            for (int q = 0; q < NW; q++) {
                if (q < wv) at += sWsum[q];
                dd += sWsum[q];
            }
            if (ok) sC[at] = x;
            __syncthreads();
        }
        if (dd < R) continue;                          // block-uniform
        if constexpr (R >= 3)
            for (int i = t; i < dd * ST; i += BT) sS[i] = 0;
        for (int i = t; i < dd; i += BT) {
            const uint32_t h = (uint32_t)sC[i] * 2654435761u, slot = 0x80000000u | ((h & 0xfffffu) << 11) | (uint32_t)i;
            uint32_t at = h >> (32 - SB);
            while (atomicCAS(&sH[at], 0u, slot) != 0u) at = (at + 1) & ((1u << SB) - 1u);
            if constexpr (R == 2) sCnt2[i] = 0;
            if constexpr (R >= 4) sCnt64[i] = 0;
        }
        __syncthreads();
        u64 hits = 0;
        for (int c0 = 0; c0 < dd; c0 += WAVE) {
            // 64 members' out-lists: a lane holds one's start and length
            const int32_t x = sC[min(c0 + L, dd - 1)];
            const int64_t o0 = dag_off[x];
            const int32_t ln = (int32_t)(row_ptr[x + 1] - o0);
            for (int mi = wv; mi < WAVE && c0 + mi < dd; mi += NW) {
                const int i = c0 + mi;
                const int32_t len = __builtin_amdgcn_readlane(ln, mi);
                const uint32_t plo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)o0, mi);
                const uint32_t phi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((u64)o0 >> 32), mi);
                const int32_t *list = col + (int64_t)(((u64)phi << 32) | plo);
                uint32_t own = 0;
                for (int e0 = 0; e0 < len; e0 += 4 * WAVE) {
                    int32_t y[4];
                    uint32_t h[4], sl[4];
#pragma unroll
                    for (int u = 0; u < 4; u++) y[u] = list[min(e0 + u * WAVE + L, len - 1)];
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        h[u] = (uint32_t)y[u] * 2654435761u;
                        sl[u] = sH[h[u] >> (32 - SB)];
                    }
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        if (e0 + u * WAVE >= len) break;
                        uint32_t s = e0 + u * WAVE + L < len ? sl[u] : 0u, at = h[u] >> (32 - SB);
                        const uint32_t tag = 0x100000u | (h[u] & 0xfffffu);
                        int j = -1;
                        while (s) {
                            if ((s >> 11) == tag && sC[s & 0x7ffu] == y[u]) {
                                j = (int)(s & 0x7ffu);
                                break;
                            }
                            at = (at + 1) & ((1u << SB) - 1u);
                            s = sH[at];
                        }
                        if (j >= 0) {
                            if constexpr (R == 2) {
                                atomicAdd(&sCnt2[j], 1u);
                                own++;
                            } else {
                                atomicOr((unsigned long long *)&sS[i * ST + (j >> 6)], 1ull << (j & 63));
                                atomicOr((unsigned long long *)&sS[j * ST + (i >> 6)], 1ull << (i & 63));
                            }
                        }
                    }
                }
                if constexpr (R == 2) {
                    own = wave_sum(own);
                    hits += own;
                    if (L == 0 && own) atomicAdd(&sCnt2[i], own);
                }
            }
        }
        __syncthreads();
        u64 tot = 0;                                   // members' counts, each clique once for each of its R members
        if constexpr (R == 3) {
            for (int i = t; i < dd; i += BT) cnt[i] = 0;
            __syncthreads();
            for (int J = wv; J * 32 < dd; J += NW) tri_block<(CAP + 63) / 64 * 2>(J, dd, sS, ST, cnt);
        } else if constexpr (R == 4) {
            int qn = 0;
            uint32_t *qu = sQ[wv];
            for (int i = wv; i < dd; i += NW) {
                const u64 mine = sS[i * ST + min(L, W - 1)];
                for (int q = i >> 6; q < W; q++) {
                    u64 m = __shfl(mine, q, WAVE);
                    if (q == (i >> 6)) m &= (i & 63) == 63 ? 0ull : (~0ull << ((i & 63) + 1));
                    if (!m) continue;                  // wave-uniform
                    if ((m >> L) & 1ull) qu[qn + __popcll(m & lanemask_lt())] = ((uint32_t)i << 16) | (uint32_t)(q * 64 + L);
                    qn += __popcll(m);
                    __builtin_amdgcn_wave_barrier();
                    if (qn >= WAVE) {
                        quad_drain<W>(qu, WAVE, sS, ST, sCnt64);
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
            if (qn) quad_drain<W>(qu, qn, sS, ST, sCnt64);
        }
        __syncthreads();
        for (int i = t; i < dd; i += BT) {
            u64 c;
            if constexpr (R == 2) c = sCnt2[i];
            else if constexpr (R == 3) c = cnt[i] / 2;
            else c = sCnt64[i] / 3;
            if (c) ctx.add(sC[i], c);
            if constexpr (R >= 3) tot += c;
        }
        if constexpr (R == 2) tot = L == 0 ? 2 * hits : 0;
        tot = wave_sum(tot);
        if (L == 0) sTot[wv] = tot;
        __syncthreads();
        if (t == 0) {
            u64 s = 0;
            for (int q = 0; q < NW; q++) s += sTot[q];
            if (s) ctx.add_prefix(it, s / (u64)R);
        }
        __syncthreads();
    }
}

// ---- huge engine for R == 2 (any |N+(w)|): global binary searches ----------
template <class Ctx>
__global__ __launch_bounds__(BLOCK) void k_engine_huge_r2(Ctx ctx, const int64_t *row_ptr, const int32_t *col,
                                                          const int64_t *dag_off, int64_t nitems,
                                                          const int32_t *nitems_dev) {
    if (nitems_dev) nitems = *nitems_dev;
    __shared__ u64 sTot[WAVES_PER_BLOCK];
    for (int64_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const int32_t w = ctx.root(it);
        const int64_t s0 = dag_off[w], e0 = row_ptr[w + 1];
        const int64_t d = e0 - s0;
        u64 tot = 0;
        for (int64_t i = threadIdx.x; i < d; i += BLOCK) {
            int32_t x = col[s0 + i];
            if (!ctx.accept(it, x)) continue;
            u64 cx = 0;
            for (int64_t e = dag_off[x]; e < row_ptr[x + 1]; e++) {
                int32_t y = col[e];
                if (!ctx.accept(it, y)) continue;
                if (bsearch_i32(col, s0, e0, y) >= 0) {
                    ctx.add(y, 1);
                    cx++;
                }
            }
            if (cx) ctx.add(x, cx);
            tot += cx;
        }
        tot = wave_sum(tot);
        if (lane() == 0) sTot[threadIdx.x / WAVE] = tot;
        __syncthreads();
        if (threadIdx.x == 0) {
            u64 t = 0;
            for (int i = 0; i < WAVES_PER_BLOCK; i++) t += sTot[i];
            if (t) ctx.add_prefix(it, t);
        }
        __syncthreads();
    }
}

}  // namespace dsd
