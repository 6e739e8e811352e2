// K1 (CSR build) and K2 (degree-ordered DAG orientation).
//
// The paper's data model is a simple undirected graph (Section 3).  Raw pairs
// are canonicalised to (min, max) keys, radix-sorted and de-duplicated; the
// degree order (deg, id) ascending gives every vertex a rank; the edges are
// re-keyed in rank space in both directions and sorted again, which yields a
// CSR whose rows are sorted by rank.  The out-neighbours of r in the DAG
// u -> v iff (deg u, u) < (deg v, v) are then the tail of row r.  Listing
// each clique from its lowest-rank member is the ordered enumeration the
// paper borrows for Algorithm 3 (Section 5.3); the degree order keeps the
// out-degrees small.
#include <algorithm>

#include "graph.hpp"

namespace dsd {

static int bits_for(int64_t n) {
    int b = 1;
    while (((int64_t)1 << b) - 1 < n) b++;
    return b;   // n <= 2^b - 1, so every id < 2^b - 1
}

__global__ void k_pair_keys(const int32_t *src, const int32_t *dst, int64_t P, int32_t n, int bits, u64 *keys,
                            int32_t *bad) {
    const u64 invalid = (bits >= 32) ? ~0ull : ((1ull << (2 * bits)) - 1ull);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t u = src[i], v = dst[i];
        if (u < 0 || u >= n || v < 0 || v >= n) {
            *bad = 1;
            keys[i] = invalid;
            continue;
        }
        if (u == v) { keys[i] = invalid; continue; }
        u64 a = (u64)(u < v ? u : v), b = (u64)(u < v ? v : u);
        keys[i] = (a << bits) | b;
    }
}

// flags[i] = 1 if keys[i] is a valid key that differs from its predecessor
__global__ void k_unique_flags(const u64 *keys, int64_t P, u64 invalid, int64_t *flags) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        u64 k = keys[i];
        flags[i] = (k != invalid && (i == 0 || keys[i - 1] != k)) ? 1 : 0;
    }
}

__global__ void k_unique_compact(const u64 *keys, int64_t P, u64 invalid, const int64_t *pos, u64 *out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
        u64 k = keys[i];
        if (k != invalid && (i == 0 || keys[i - 1] != k)) out[pos[i]] = k;
    }
}

__global__ void k_edge_degrees(const u64 *edges, int64_t m, int bits, int32_t *deg) {
    const u64 mask = (1ull << bits) - 1ull;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        u64 k = edges[i];
        atomicAdd(&deg[(int32_t)(k >> bits)], 1);
        atomicAdd(&deg[(int32_t)(k & mask)], 1);
    }
}

// Degrees of a large edge list.  Device-wide atomics run at about 16 G/s on
// this part whatever their addresses (8.1 ms for the 128 M ends of R-MAT
// scale 22, 64 M edges, n = 2^22), so from DEG_RANGE_EDGES edges on the ends
// are counted in LDS instead: the edges are sorted by their lower end a, one
// more radix pass groups a copy of them by the top 8 bits of the upper end b,
// and a workgroup counts both ends that fall into one of the 256 id ranges (at most
// 2^15 counters, 128 KB) and stores the counts plainly.  Bound by reading the
// keys: 1.1 ms with the extra pass on the same graph.  A range with more than
// DEG_PART ends (ids in hub order) is split over workgroups, which then add
// their counts atomically.
constexpr int DEG_BLOCK = 1024;
constexpr int DEG_MAX_BITS = 23;                    // 2^(bits - 8) counters fit the LDS
constexpr int64_t DEG_PART = (int64_t)1 << 20;
constexpr int DEG_MAX_PARTS = 16;
// below this the extra launches (about 25 us) cost more than the atomics
constexpr int64_t DEG_RANGE_EDGES = (int64_t)1 << 18;

__device__ __forceinline__ int64_t first_key_ge(const u64 *keys, int64_t m, u64 x) {
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// by_a: keys sorted ascending; by_b: the same keys grouped by the top 8 bits
// of their low half, group q starting at start_b[q * tiles] (the radix pass's
// offsets of its first tile).  deg is zero on entry.
__global__ __launch_bounds__(DEG_BLOCK) void k_range_degrees(const u64 *by_a, const u64 *by_b, int64_t m, int bits,
                                                             int32_t n, const uint32_t *start_b, int64_t tiles,
                                                             int32_t *deg) {
    __shared__ int32_t cnt[1 << (DEG_MAX_BITS - 8)];
    const int q = blockIdx.x, sh = bits - 8;
    const int32_t range = 1 << sh, v0 = q << sh;
    if (v0 >= n) return;
    const int64_t a0 = first_key_ge(by_a, m, (u64)q << (sh + bits));
    const int64_t a1 = q == 255 ? m : first_key_ge(by_a, m, (u64)(q + 1) << (sh + bits));
    const int64_t b0 = start_b[(int64_t)q * tiles], b1 = q == 255 ? m : start_b[(int64_t)(q + 1) * tiles];
    const int64_t ends = (a1 - a0) + (b1 - b0);
    const int parts = (int)min((int64_t)DEG_MAX_PARTS, ends / DEG_PART + 1), part = blockIdx.y;
    if (part >= parts) return;
    for (int i = threadIdx.x; i < range; i += DEG_BLOCK) cnt[i] = 0;
    __syncthreads();
    const int64_t step = (int64_t)parts * DEG_BLOCK, first = (int64_t)part * DEG_BLOCK + threadIdx.x;
    for (int64_t i = a0 + first; i < a1; i += step) atomicAdd(&cnt[(int32_t)(by_a[i] >> bits) - v0], 1);
    const u64 mask = (1ull << bits) - 1ull;
    for (int64_t i = b0 + first; i < b1; i += step) atomicAdd(&cnt[(int32_t)(by_b[i] & mask) - v0], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < range && v0 + i < n; i += DEG_BLOCK) {
        if (parts == 1) deg[v0 + i] = cnt[i];
        else if (cnt[i]) atomicAdd(&deg[v0 + i], cnt[i]);
    }
}

__global__ void k_rank_keys(const int32_t *deg, int32_t n, int bits, u64 *keys) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        keys[v] = ((u64)deg[v] << bits) | (u64)v;
}

// ranks, and every row's length (the degree in the sorted key)
__global__ void k_rank_perm(const u64 *keys, int32_t n, int bits, int32_t *orig_of, int32_t *rank_of,
                            int64_t *row_len) {
    const u64 mask = (1ull << bits) - 1ull;
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        int32_t v = (int32_t)(keys[r] & mask);
        orig_of[r] = v;
        rank_of[v] = (int32_t)r;
        row_len[r] = (int64_t)(keys[r] >> bits);
    }
}

// K2: re-key every edge in rank space, both directions
__global__ void k_orient_keys(const u64 *edges, int64_t m, int bits, const int32_t *rank_of, u64 *keys) {
    const u64 mask = (1ull << bits) - 1ull;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        u64 k = edges[i];
        u64 ru = (u64)rank_of[(int32_t)(k >> bits)];
        u64 rv = (u64)rank_of[(int32_t)(k & mask)];
        keys[2 * i] = (ru << bits) | rv;
        keys[2 * i + 1] = (rv << bits) | ru;
    }
}

// col from the sorted keys (the row starts come from a scan of the row
// lengths: filling them from the row boundaries leaves every isolated vertex
// before the first row to one thread, 48 of 69 ms at R-MAT scale 22), and the
// end of the last row
__global__ void k_csr_cols(const u64 *keys, int64_t E, int32_t n, int bits, int32_t *col, int64_t *row_ptr) {
    const u64 mask = (1ull << bits) - 1ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) row_ptr[n] = E;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < E; i += (int64_t)gridDim.x * blockDim.x)
        col[i] = (int32_t)(keys[i] & mask);
}

// dag_off[r] = first position of row r holding a rank > r; the largest
// degrees, and the wedge sums w2 and s2 (out: maxes in [0, 2), sums in
// [0, 2)).  Each workgroup reduces before its four atomics: one per wave from
// 32,768 waves queued on the same addresses for 1.1 ms at n = 2^22.
constexpr int DAG_GRID = 1024;
__global__ __launch_bounds__(BLOCK) void k_dag_off(const int64_t *row_ptr, const int32_t *col, int32_t n,
                                                   int64_t *dag_off, int32_t *maxes, u64 *sums) {
    __shared__ int32_t sMd[WAVES_PER_BLOCK], sMo[WAVES_PER_BLOCK];
    __shared__ u64 sW2[WAVES_PER_BLOCK], sS2[WAVES_PER_BLOCK];
    int32_t md = 0, mo = 0;
    u64 w2 = 0, s2 = 0;
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s0 = row_ptr[r], e = row_ptr[r + 1];
        int64_t lo = s0, hi = e;
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if (col[mid] > (int32_t)r) hi = mid; else lo = mid + 1;
        }
        dag_off[r] = lo;
        const int32_t d = (int32_t)(e - s0), o = (int32_t)(e - lo);
        md = d > md ? d : md;
        mo = o > mo ? o : mo;
        w2 += (u64)(d - o) * (u64)o;
        s2 += (u64)d * (u64)o;
    }
    md = wave_max(md);
    mo = wave_max(mo);
    w2 = wave_sum(w2);
    s2 = wave_sum(s2);
    const int wv = threadIdx.x / WAVE;
    if (lane() == 0) {
        sMd[wv] = md;
        sMo[wv] = mo;
        sW2[wv] = w2;
        sS2[wv] = s2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < WAVES_PER_BLOCK; i++) {
            md = max(md, sMd[i]);
            mo = max(mo, sMo[i]);
            w2 += sW2[i];
            s2 += sS2[i];
        }
        atomicMax(&maxes[0], md);
        atomicMax(&maxes[1], mo);
        atomicAdd(&sums[0], w2);
        atomicAdd(&sums[1], s2);
    }
}

void build_graph(int32_t n, int64_t P, const int32_t *src, const int32_t *dst, DevGraph &g, hipStream_t s,
                 Scratch &sc, float *t_orient_ms, Scratch *keep) {
    g.n = n;
    g.bits = bits_for(n > 0 ? n : 1);
    const int bits = g.bits;
    const u64 invalid = (bits >= 32) ? ~0ull : ((1ull << (2 * bits)) - 1ull);
    int64_t m = 0;
    int32_t *d_bad = sc.get_n<int32_t>(4);
    fill_i32(d_bad, 0, 4, s);
    u64 *edges = nullptr, *spare = nullptr;   // unique keys; a second buffer of their size
    if (P > 0) {
        u64 *keys = sc.get_n<u64>(P), *tmp = sc.get_n<u64>(P);
        k_pair_keys<<<grid_for(P, BLOCK, 8192), BLOCK, 0, s>>>(src, dst, P, n, bits, keys, d_bad);
        radix_sort_u64(keys, tmp, P, 2 * bits, s, sc);
        int64_t *pos = sc.get_n<int64_t>(P);
        k_unique_flags<<<grid_for(P, BLOCK, 8192), BLOCK, 0, s>>>(keys, P, invalid, pos);
        scan_exclusive_i64(pos, pos, P, s, sc);
        int64_t last_pos = 0;
        u64 last_key = 0, prev_key = 0;
        int32_t bad = 0;
        Readback rb(sc);
        rb.add(&last_pos, pos + P - 1).add(&last_key, keys + P - 1).add(&bad, d_bad);
        if (P > 1) rb.add(&prev_key, keys + P - 2);
        rb.run(s);
        if (bad) throw Error(-1, "vertex id outside [0, n)");
        m = last_pos + ((last_key != invalid && (P == 1 || prev_key != last_key)) ? 1 : 0);
        edges = tmp;   // reuse: unique keys
        spare = keys;
        if (m > 0) k_unique_compact<<<grid_for(P, BLOCK, 8192), BLOCK, 0, s>>>(keys, P, invalid, pos, edges);
    }
    g.m = m;
    const int64_t E = 2 * m;
    if (E > (int64_t)0x7fffffff) throw Error(-5, "more than 2^31-1 adjacency entries");
    hipEvent_t e0, e1;
    DSD_HIP(hipEventCreate(&e0));
    DSD_HIP(hipEventCreate(&e1));
    DSD_HIP(hipEventRecord(e0, s));
    // degrees in caller ids -> rank order
    int32_t *deg = sc.get_n<int32_t>(n);
    if (keep) {
        g.owned = false;
        g.row_ptr = keep->get_n<int64_t>((int64_t)n + 1);
        g.col = keep->get_n<int32_t>(E);
        g.dag_off = keep->get_n<int64_t>(n);
        g.orig_of = keep->get_n<int32_t>(n);
        g.rank_of = keep->get_n<int32_t>(n);
    } else {
        g.owned = true;
        DSD_HIP(hipMalloc(&g.row_ptr, ((size_t)n + 1) * sizeof(int64_t)));
        DSD_HIP(hipMalloc(&g.col, (size_t)(E > 0 ? E : 1) * sizeof(int32_t)));
        DSD_HIP(hipMalloc(&g.dag_off, (size_t)(n > 0 ? n : 1) * sizeof(int64_t)));
        DSD_HIP(hipMalloc(&g.orig_of, (size_t)(n > 0 ? n : 1) * sizeof(int32_t)));
        DSD_HIP(hipMalloc(&g.rank_of, (size_t)(n > 0 ? n : 1) * sizeof(int32_t)));
    }
    int32_t *maxes = d_bad + 2;
    if (n > 0) {
        fill_i32(deg, 0, n, s);
        if (m >= DEG_RANGE_EDGES && bits > 8 && bits <= DEG_MAX_BITS) {
            const int64_t tiles = radix_tiles(m);
            uint32_t *start = sc.get_n<uint32_t>(256 * tiles);
            radix_pass_u64(edges, spare, m, bits - 8, start, s, sc);
            const unsigned parts = (unsigned)std::min<int64_t>(DEG_MAX_PARTS, 2 * m / DEG_PART + 1);
            k_range_degrees<<<dim3(256, parts), DEG_BLOCK, 0, s>>>(edges, spare, m, bits, n, start, tiles, deg);
        } else if (m > 0) {
            k_edge_degrees<<<grid_for(m, BLOCK, 8192), BLOCK, 0, s>>>(edges, m, bits, deg);
        }
        u64 *rk = sc.get_n<u64>(n), *rtmp = sc.get_n<u64>(n);
        k_rank_keys<<<grid_for(n, BLOCK, 8192), BLOCK, 0, s>>>(deg, n, bits, rk);
        radix_sort_u64(rk, rtmp, n, 2 * bits, s, sc);
        k_rank_perm<<<grid_for(n, BLOCK, 8192), BLOCK, 0, s>>>(rk, n, bits, g.orig_of, g.rank_of, g.row_ptr);
        scan_exclusive_i64(g.row_ptr, g.row_ptr, n, s, sc);
    }
    u64 *k3 = nullptr;
    if (E > 0) {
        k3 = sc.get_n<u64>(E);
        u64 *t3 = sc.get_n<u64>(E);
        k_orient_keys<<<grid_for(m, BLOCK, 8192), BLOCK, 0, s>>>(edges, m, bits, g.rank_of, k3);
        radix_sort_u64(k3, t3, E, 2 * bits, s, sc);
    }
    k_csr_cols<<<grid_for(E, BLOCK, 8192), BLOCK, 0, s>>>(k3, E, n, bits, g.col, g.row_ptr);
    u64 *wed = sc.get_n<u64>(2);
    fill_u64(wed, 0, 2, s);
    if (n > 0) k_dag_off<<<grid_for(n, BLOCK, DAG_GRID), BLOCK, 0, s>>>(g.row_ptr, g.col, n, g.dag_off, maxes, wed);
    DSD_HIP(hipEventRecord(e1, s));
    int32_t hm[2] = {0, 0};
    u64 hw[2] = {0, 0};
    Readback(sc).add(hm, maxes, 2).add(hw, wed, 2).run(s);
    g.w2 = hw[0];
    g.s2 = hw[1];
    g.maxdeg = hm[0];
    g.maxdout = hm[1];
    if (t_orient_ms) DSD_HIP(hipEventElapsedTime(t_orient_ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
}

void free_graph(DevGraph &g) {
    if (g.owned) {
        (void)hipFree(g.row_ptr);
        (void)hipFree(g.col);
        (void)hipFree(g.dag_off);
        (void)hipFree(g.orig_of);
        (void)hipFree(g.rank_of);
    }
    g = DevGraph();
}

}  // namespace dsd
