// State of the round-synchronous peel shared by its round kernels (peel.hip)
// and the clique tail (ctail.hip).
#pragma once

#include "graph.hpp"

namespace dsd {

struct PeelCtl {
    int64_t n_alive;   // alive vertices over all graphs (the host polls it)
    int32_t round;
    int32_t cur;       // frontier buffer in use
    int32_t nF[2];     // frontier sizes (all graphs)
    int32_t nB[2];     // chunk items of large frontier vertices (h = 3)
    int32_t nlist[2];  // alive-list sizes
    int32_t lcur;      // alive list in use
    int32_t nsel[2];   // graphs that open a level in the round using buffer 0 / 1
    int32_t nitems[8]; // (v, w) work items per class (h >= 4)
    int64_t htop[2];   // slots handed out in the global neighbourhood hashes (h = 3)
    int64_t nW;        // wide (v, w) items of this round (h = 3)
    int32_t nT[2];     // row items of the frontier (triangle lists)
    int32_t pending;   // tail mode: a round has been started and not yet finished
    int32_t nTouch;    // x-star pattern: survivors whose degree fell this round
    int32_t nBig[2];   // h >= 4 root mode: single-workgroup items of the frontier
    u64 work[4];       // main kernel's pairs, neighbours and (h >= 4) row entries, counting kernel's bitmap
                       // words, over the whole peel (when counted)
};

// one graph of the batch (a single graph is a batch of one)
struct GraphState {
    u64 k;             // current level
    u64 kcand;         // smallest alive degree, gathered when a level opens
    u64 mu_alive;      // cliques among the graph's alive vertices
    u64 destroyed;     // cliques destroyed in this round
    u64 destroyed_m;   // root mode: per-member counts of this round's cliques (each clique h - 1 times)
    int64_t n_alive;
    int64_t lv_base;   // first entry of the graph's level table
    int32_t nF[2];     // the graph's frontier sizes
    int32_t nlevels;
    int32_t sel;       // this round opens a new level (fixed for the whole round)
};

struct PeelBufs {
    PeelCtl *ctl;
    GraphState *gs;
    const int32_t *gid;  // [n] graph of every vertex (nullptr: one graph)
    int32_t G;
    const int64_t *row_ptr;
    const int32_t *col;
    const int64_t *dag_off;
    int32_t *stamp;    // ALIVE, removal round, or -1 (not taking part)
    u64 *deg;          // current clique-degree
    u64 *core;
    int32_t *F;        // [2][n] frontiers
    int64_t *B;        // [2][bcap] (v << 32 | chunk) for frontier vertices of degree > SMALL_DEG
    int64_t bcap;
    int32_t *lists;    // [2][n] alive lists
    u64 *lv_k, *lv_size, *lv_mu;  // level tables
    int32_t *item_v, *item_w;     // [5][cap] work items (h >= 4)
    int64_t item_cap;
    int32_t *hkey;     // [2][hcap] global hashes of N(v) for large frontier vertices (h = 3)
    uint32_t *hval;
    int64_t hcap;
    int64_t *hbase;    // [n] first slot of v's hash in its round's half
    int64_t *W;        // [wcap] wide items (v << 32 | w): w with a long out-list (h = 3)
    int64_t wcap;
    int32_t n;
    int32_t h;
    const int64_t *tvoff; // triangle lists (nullptr: none): row starts, (a, b) pairs
    const int32_t *tpairs;
    int64_t *T;          // [2][tcap] row items (v << 32 | chunk) of frontier vertices
    int64_t tcap;
    int32_t pattern;     // 0: cliques; 1: x-stars with px tails; 2: 4-loops
    int32_t px;
    int32_t *ydeg;       // x-star: residual degree, now and at the start of the round
    int32_t *yold;
    int32_t *tround;     // x-star: round in which the vertex's degree last fell
    int32_t *touch;      // x-star: this round's survivors whose degree fell
    int32_t *lkey;       // 4-loop: [blocks][lsize] hash of a frontier vertex's 2-hop neighbours
    uint32_t *lval;
    int64_t lsize;
    int32_t count_work;  // the main kernel adds up its pairs and neighbours
    int32_t minpeel;     // min-degree mode: every round removes the minimum-degree vertices
    const u64 *eset;     // h >= 4: open-addressing set of the edges among the peel's vertices
    int32_t eset_bits;   // (2^eset_bits slots, keys (lo << 32 | hi) in rank space)
    int32_t rootmode;    // h >= 4: the frontier vertices' own cliques (k_root_edges / k_root_count)
    int64_t *Big;        // [2][bigcap] root mode: (v << 32 | chunk) single-workgroup items
    int64_t bigcap;
    u64 *rbits;          // [2][rcap] root mode: bitmap rows of the sliced vertices' neighbourhoods
    int64_t rcap;
    int64_t *rbase;      // [n] first word of v's region in its round's half
};

// ---- the clique tail (ctail.hip): the rest of an h >= 4 peel ----
// Finishes the peel of b's graphs (between two rounds) once their alive
// vertices are few enough for adjacency bitmaps; min_degree as in peel().
// Returns false, having changed nothing, when they are not (or with
// DSD_TAIL_ENGINE=0).  CT_ROUND_CYCLES: up to these its workgroup keeps a
// round to itself.
constexpr int64_t CT_ROUND_CYCLES = 100000;
constexpr int64_t CT_MAX = 131072;             // alive vertices per graph (2,048-word rows: live sets of 16 KB in LDS)
constexpr int64_t CT_MATRIX_WORDS = (int64_t)1 << 29;   // all matrices together (4 GiB)
constexpr int64_t CT_VERTICES = (int64_t)1 << 23;       // vertices of all graphs together (items fit the counter)
bool clique_tail(const PeelBufs &b, int h, int64_t n_alive, hipStream_t s, Scratch &sc, KernelTimes *kt);

}  // namespace dsd
