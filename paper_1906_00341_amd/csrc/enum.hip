// K3: clique-degrees (Definition 3) on the degree-ordered DAG.
//
// Every h-clique is listed once, from its lowest-rank member r: the other
// h-1 members form an (h-1)-clique of the sub-DAG induced on N+(r).  Roots
// are binned by out-degree into a wave class (one wave per root, |N+| <= 64)
// and block classes (one workgroup per root, candidate set, hash and bitmap
// staged in LDS); each root flushes at most |N+(r)| + 1 global 64-bit atomics.
#include <algorithm>
#include <cctype>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>

#include "engine.hpp"
#include "graph.hpp"

namespace dsd {

struct EnumCtx {
    const int32_t *roots;
    const uint8_t *mask;
    u64 *deg;
    __device__ __forceinline__ int32_t root(int64_t it) const { return roots[it]; }
    __device__ __forceinline__ bool accept(int64_t, int32_t x) const { return mask == nullptr || mask[x] != 0; }
    __device__ __forceinline__ void add(int32_t x, u64 c) const { atomic_add_u64(&deg[x], c); }
    __device__ __forceinline__ void add_prefix(int64_t it, u64 t) const { atomic_add_u64(&deg[roots[it]], t); }
};

// h = 2: the clique-degree is the degree (inside the mask: one wave per
// vertex, since a hub's row is long)
__global__ void k_deg_h2(const int64_t *row_ptr, int32_t n, u64 *deg) {
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        deg[v] = (u64)(row_ptr[v + 1] - row_ptr[v]);
}

__global__ __launch_bounds__(BLOCK) void k_deg_h2_masked(const int64_t *row_ptr, const int32_t *col,
                                                          const uint8_t *mask, int32_t n, u64 *deg) {
    const int wv = threadIdx.x / WAVE;
    for (int64_t v = (int64_t)blockIdx.x * WAVES_PER_BLOCK + wv; v < n; v += (int64_t)gridDim.x * WAVES_PER_BLOCK) {
        u64 c = 0;
        if (mask[v])
            for (int64_t e = row_ptr[v] + lane(); e < row_ptr[v + 1]; e += WAVE) c += mask[col[e]] ? 1 : 0;
        c = wave_sum(c);
        if (lane() == 0) deg[v] = c;
    }
}

__device__ __forceinline__ u64 binom_sat_dev(u64 x, int r) {
    if ((u64)r > x) return 0;
    unsigned __int128 acc = 1;
    for (int i = 1; i <= r; i++) {
        acc = acc * (unsigned __int128)(x - (u64)r + (u64)i) / (unsigned __int128)i;
        if (acc > (unsigned __int128)~0ull) return ~0ull;
    }
    return (u64)acc;
}

// Roots are binned by out-degree.  The bins up to 768 (R = 2: 2,048), and up
// to 1,088 for R = 3, hold what k_engine_rows keeps in LDS: 257-512 apart from
// 513-768 so that three workgroups fit a CU, 1,088 because 17-word rows are the
// longest that fit beside the table (148 KB).  Beyond, the bitmap lives in
// global memory.  A launch class (what the tuning calls a class) is one bin
// or two neighbouring ones.
constexpr int NBIN = 8;
// first bin of every launch class, and the end
__host__ __device__ constexpr int class_bin(int R, int c) {
    return R <= 2 ? c : c <= 2 ? c : c == 3 ? 4 : c == 4 ? 6 : 7;
}

// bin of a root by its out-degree; -1 = no clique can be rooted here
__device__ __forceinline__ int root_bin(int d, int R) {
    if (d < R) return -1;
    if (d <= 64) return 0;
    if (R <= 2) return d <= 2048 ? 1 : 2;
    if (d <= 256) return 1;
    if (d <= 512) return 2;
    if (d <= 768) return 3;
    if (d <= 1088 && R == 3) return 4;
    if (d <= 1280) return 5;
    if (d <= 2048) return 6;
    return 7;   // beyond the bitmap kernels
}

__device__ __forceinline__ u64 sat_add(u64 a, u64 b) { return (a + b < a) ? ~0ull : a + b; }

// clears what a call counts into: the degrees, the bins' two counters and the bound
__global__ void k_enum_init(u64 *deg, int64_t n, int32_t *cursor, u64 *bound) {
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * blockDim.x) deg[i] = 0;
    if (i0 < 2 * NBIN) cursor[i0] = 0;
    if (i0 == 0) *bound = 0;
}

struct RootOffsets {
    int32_t off[NBIN + 1];
};
constexpr int CLASSIFY_PER = 16;                          // roots per thread
constexpr int CLASSIFY_TILE = BLOCK * CLASSIFY_PER;       // consecutive roots per workgroup

// FILL false: per-bin counts and a saturating bound sum_r C(d+(r), R) on the
// number of cliques; FILL true: the bins' lists, from off on.  The bins are
// counted in LDS, so that a workgroup pays one global atomic per bin for its
// 4,096 roots (one per bin and wave: 0.31 ms each pass for 2^22 roots).
template <bool FILL>
__global__ __launch_bounds__(BLOCK) void k_classify(const int64_t *row_ptr, const int64_t *dag_off, const uint8_t *mask,
                                                    int32_t n, int R, int32_t *cursor, int32_t *lists, RootOffsets off,
                                                    u64 *bound) {
    __shared__ int32_t sCnt[NBIN];
    __shared__ u64 sBound[WAVES_PER_BLOCK];
    static_assert(NBIN <= 15, "a bin has to fit four bits");
    if (threadIdx.x < NBIN) sCnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * CLASSIFY_TILE + threadIdx.x;
    u64 b = 0, bins = 0;   // a thread's bins, four bits each (15: no root)
#pragma unroll 4
    for (int j = 0; j < CLASSIFY_PER; j++) {
        const int64_t r = r0 + (int64_t)j * BLOCK;
        int c = -1;
        if (r < n && (!mask || mask[r])) {
            const int d = (int)(row_ptr[r + 1] - dag_off[r]);
            c = root_bin(d, R);
            if (!FILL && c >= 0) b = sat_add(b, binom_sat_dev((u64)d, R));
        }
        bins |= (u64)(c & 15) << (4 * j);
        for (int k = 0; k < NBIN; k++) {
            const u64 m = __ballot(c == k);
            if (m && lane() == 0) atomicAdd(&sCnt[k], __popcll(m));
        }
    }
    if (!FILL) {
        for (int d = WAVE / 2; d > 0; d >>= 1) b = sat_add(b, __shfl_xor(b, d, WAVE));
        if (lane() == 0) sBound[threadIdx.x / WAVE] = b;
    }
    __syncthreads();
    if (threadIdx.x < NBIN && sCnt[threadIdx.x])
        sCnt[threadIdx.x] = atomicAdd(&cursor[threadIdx.x], sCnt[threadIdx.x]);
    if (!FILL) {
        if (threadIdx.x) return;
        for (int w = 1; w < WAVES_PER_BLOCK; w++) b = sat_add(b, sBound[w]);
        if (b) {
            const u64 old = atomicAdd(bound, b);
            if (old + b < old) atomicExch(bound, ~0ull);
        }
        return;
    }
    __syncthreads();
    for (int j = 0; j < CLASSIFY_PER; j++) {
        const int c = (int)(bins >> (4 * j) & 15);
        for (int k = 0; k < NBIN; k++) {
            const u64 m = __ballot(c == k);
            if (!m) continue;
            int32_t base = 0;
            if (lane() == 0) base = atomicAdd(&sCnt[k], __popcll(m));
            base = __shfl(base, 0, WAVE);
            if (c == k) lists[off.off[k] + base + __popcll(m & lanemask_lt())] = (int32_t)(r0 + (int64_t)j * BLOCK);
        }
    }
}

// ---------------------------------------------------------------- launch grids and their tuning
//
// Each out-degree class of roots is one launch whose grid is capped: the
// workgroups loop over the class's roots, so the cap trades occupancy and
// tail balance against per-workgroup start-up (and, for the classes whose
// bitmaps live in global memory, scratch).  The caps below are the
// defaults; dsd_autotune times a set of caps per class on a caller's graph
// and keeps the fastest in a process-wide table keyed by (architecture, h,
// class), which dsd_tune_load (or DSD_TUNE_FILE, read once) fills from a
// JSON file and dsd_autotune can write back.

static int default_cap(int R, int c) {
    if (c == 0) return 8192;
    if (R <= 2) return c == 1 ? 4096 : 1024;
    return c == 1 ? 4096 : c == 2 ? 2048 : 512;
}

struct TuneTable {
    std::mutex mu;
    std::map<std::string, int> cap;
    bool env_read = false;
};
static TuneTable &tune_table() {
    static TuneTable *t = new TuneTable();   // never destroyed: launches may run during static destruction
    return *t;
}

// the current device's architecture, e.g. gfx950 (the name up to its feature suffix)
static std::string arch_name() {
    static std::mutex mu;
    static std::map<int, std::string> names;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return "unknown";
    std::lock_guard<std::mutex> lk(mu);
    auto it = names.find(dev);
    if (it != names.end()) return it->second;
    hipDeviceProp_t p;
    std::string a = "unknown";
    if (hipGetDeviceProperties(&p, dev) == hipSuccess) {
        a = p.gcnArchName;
        const size_t colon = a.find(':');
        if (colon != std::string::npos) a = a.substr(0, colon);
    }
    names[dev] = a;
    return a;
}

static std::string tune_key(const std::string &arch, int h, int c) {
    return arch + "/h" + std::to_string(h) + "/c" + std::to_string(c);
}

// the JSON file: one flat object, "gfx950/h4/c2": 1024, ...
static void tune_parse(const std::string &text, std::map<std::string, int> &out) {
    size_t i = 0;
    auto ws = [&] {
        while (i < text.size() && std::isspace((unsigned char)text[i])) i++;
    };
    auto bad = [] { throw Error(-1, "tuning file is not a flat JSON object of \"key\": integer pairs"); };
    ws();
    if (i >= text.size() || text[i] != '{') bad();
    i++;
    ws();
    if (i < text.size() && text[i] == '}') return;
    while (true) {
        ws();
        if (i >= text.size() || text[i] != '"') bad();
        const size_t k0 = ++i;
        while (i < text.size() && text[i] != '"') i++;
        if (i >= text.size()) bad();
        const std::string key = text.substr(k0, i - k0);
        i++;
        ws();
        if (i >= text.size() || text[i] != ':') bad();
        i++;
        ws();
        const size_t v0 = i;
        while (i < text.size() && std::isdigit((unsigned char)text[i])) i++;
        if (i == v0 || i - v0 > 9) bad();
        const int v = std::atoi(text.substr(v0, i - v0).c_str());
        if (v < 1 || v > 65536) bad();
        out[key] = v;
        ws();
        if (i < text.size() && text[i] == ',') {
            i++;
            continue;
        }
        if (i < text.size() && text[i] == '}') break;
        bad();
    }
}

void tune_load(const char *path) {
    std::map<std::string, int> m;
    if (path) {
        FILE *f = std::fopen(path, "rb");
        if (!f) throw Error(-1, std::string("cannot open tuning file ") + path);
        std::string text;
        char buf[4096];
        size_t got;
        while ((got = std::fread(buf, 1, sizeof(buf), f)) > 0) text.append(buf, got);
        std::fclose(f);
        tune_parse(text, m);
    }
    TuneTable &t = tune_table();
    std::lock_guard<std::mutex> lk(t.mu);
    t.cap = m;
    t.env_read = true;
}

static void tune_save(const char *path) {
    std::map<std::string, int> m;
    if (FILE *f = std::fopen(path, "rb")) {
        std::string text;
        char buf[4096];
        size_t got;
        while ((got = std::fread(buf, 1, sizeof(buf), f)) > 0) text.append(buf, got);
        std::fclose(f);
        try {
            tune_parse(text, m);
        } catch (const Error &) {
            m.clear();   // an unreadable old file is replaced
        }
    }
    TuneTable &t = tune_table();
    {
        std::lock_guard<std::mutex> lk(t.mu);
        for (auto &kv : t.cap) m[kv.first] = kv.second;
    }
    const std::string tmp = std::string(path) + ".tmp";
    FILE *f = std::fopen(tmp.c_str(), "wb");
    if (!f) throw Error(-1, std::string("cannot write tuning file ") + path);
    std::fprintf(f, "{");
    bool first = true;
    for (auto &kv : m) {
        std::fprintf(f, "%s\n  \"%s\": %d", first ? "" : ",", kv.first.c_str(), kv.second);
        first = false;
    }
    std::fprintf(f, "\n}\n");
    const bool ok = std::fclose(f) == 0;
    if (!ok || std::rename(tmp.c_str(), path) != 0) throw Error(-1, std::string("cannot write tuning file ") + path);
}

// the grid cap of class c for R = h - 1: the tuned one, else the default
static int class_cap(int R, int c) {
    TuneTable &t = tune_table();
    std::lock_guard<std::mutex> lk(t.mu);
    if (!t.env_read) {
        t.env_read = true;
        if (const char *e = std::getenv("DSD_TUNE_FILE")) {
            std::map<std::string, int> m;
            if (FILE *f = std::fopen(e, "rb")) {
                std::string text;
                char buf[4096];
                size_t got;
                while ((got = std::fread(buf, 1, sizeof(buf), f)) > 0) text.append(buf, got);
                std::fclose(f);
                try {
                    tune_parse(text, m);
                } catch (const Error &) {
                    m.clear();   // a malformed file leaves the defaults
                }
            }
            t.cap = m;
        }
    }
    if (t.cap.empty()) return default_cap(R, c);
    auto it = t.cap.find(tune_key(arch_name(), R + 1, c));
    return it == t.cap.end() ? default_cap(R, c) : it->second;
}

// one bin's launch; cap: its grid cap (gs_blocks bounds the global-bitmap bins)
template <int R>
static void launch_bin(int c, int cap, const DevGraph &g, const EnumCtx &base, const int32_t *lists,
                       const int32_t *off, const int32_t *cnt, hipStream_t s, Scratch &sc, int gs_blocks) {
    if (!cnt[c]) return;
    EnumCtx ctx = base;
    ctx.roots = lists + off[c];
    const int blocks = grid_for(cnt[c], 1, cap);
    if (c == 0) {
        k_engine_wave<R, EnumCtx><<<grid_for(cnt[0], WAVES_PER_BLOCK, cap), BLOCK, 0, s>>>(ctx, g.row_ptr, g.col,
                                                                                         g.dag_off, cnt[0], nullptr);
        return;
    }
    if constexpr (R <= 2) {
        if (c == 1)
            k_engine_rows<R, 2048, 12, 1, 256, EnumCtx><<<blocks, 256, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off, cnt[1]);
        else
            k_engine_huge_r2<EnumCtx><<<blocks, BLOCK, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off, cnt[2], nullptr);
    } else {
        const int gblocks = std::min(blocks, gs_blocks);
        if (c == 1) {
            if constexpr (R <= 4)
                k_engine_rows<R, 256, 10, 4, 256, EnumCtx><<<blocks, 256, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off, cnt[1]);
            else
                k_engine_block<R, 256, 9, 4, false, EnumCtx><<<blocks, BLOCK, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                       cnt[1], nullptr, nullptr);
        } else if (c == 2) {
            if constexpr (R <= 4)
                k_engine_rows<R, 512, 11, 8, 256, EnumCtx><<<blocks, 256, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off, cnt[2]);
            else
                k_engine_block<R, 512, 11, 8, false, EnumCtx><<<blocks, BLOCK, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                        cnt[2], nullptr, nullptr);
        } else if (c == 3) {
            if constexpr (R <= 4)
                k_engine_rows<R, 768, 12, 12, 512, EnumCtx><<<blocks, 512, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                    cnt[3]);
            else
                k_engine_block<R, 768, 11, 12, false, EnumCtx><<<blocks, BLOCK, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                         cnt[3], nullptr, nullptr);
        } else if (c == 4) {
            if constexpr (R == 3)
                k_engine_rows<R, 1088, 11, 17, 512, EnumCtx><<<blocks, 512, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                     cnt[4]);
        } else if (c == 5) {
            u64 *gS = sc.get_n<u64>((int64_t)gblocks * 1280 * 20);
            k_engine_block<R, 1280, 12, 20, true, EnumCtx><<<gblocks, BLOCK, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                      cnt[5], nullptr, gS);
        } else if (c == 6) {
            // hubs of out-degree 1281..2048: 32-word bitmap rows in global memory
            u64 *gS = sc.get_n<u64>((int64_t)gblocks * 2048 * 32);
            k_engine_block<R, 2048, 12, 32, true, EnumCtx><<<gblocks, BLOCK, 0, s>>>(ctx, g.row_ptr, g.col, g.dag_off,
                                                                                      cnt[6], nullptr, gS);
        }
    }
}

// one class's launches
template <int R>
static void launch_class(int c, int cap, const DevGraph &g, const EnumCtx &base, const int32_t *lists,
                         const int32_t *off, const int32_t *cnt, hipStream_t s, Scratch &sc, int gs_blocks) {
    for (int k = class_bin(R, c); k < class_bin(R, c + 1); k++)
        launch_bin<R>(k, cap, g, base, lists, off, cnt, s, sc, gs_blocks);
}

// roots of launch class c
static int32_t class_roots(int R, int c, const int32_t *cnt) {
    int32_t n = 0;
    for (int k = class_bin(R, c); k < class_bin(R, c + 1); k++) n += cnt[k];
    return n;
}

static int nclass_of(int R) { return R <= 2 ? 3 : 5; }

template <int R>
static void launch_engine(const DevGraph &g, const EnumCtx &base, const int32_t *lists, const int32_t *off,
                          const int32_t *cnt, hipStream_t s, Scratch &sc, int gs_blocks) {
    for (int c = 0; c < nclass_of(R); c++)
        if (class_roots(R, c, cnt)) launch_class<R>(c, class_cap(R, c), g, base, lists, off, cnt, s, sc, gs_blocks);
}

static void launch_one_class(int R, int c, int cap, const DevGraph &g, const EnumCtx &ctx, const int32_t *lists,
                             const int32_t *off, const int32_t *cnt, hipStream_t s, Scratch &sc) {
    switch (R) {
        case 2: launch_class<2>(c, cap, g, ctx, lists, off, cnt, s, sc, 1 << 20); break;
        case 3: launch_class<3>(c, cap, g, ctx, lists, off, cnt, s, sc, 1 << 20); break;
        case 4: launch_class<4>(c, cap, g, ctx, lists, off, cnt, s, sc, 1 << 20); break;
        case 5: launch_class<5>(c, cap, g, ctx, lists, off, cnt, s, sc, 1 << 20); break;
        default: throw Error(-1, "h outside [2, 6]");
    }
}

// roots binned by class, deg (length n) cleared; false if the counts could
// overflow 64 bits
struct RootClasses {
    int32_t hc[NBIN];
    int32_t off[NBIN + 1];
    int32_t *lists = nullptr;
};
static bool classify_roots(const DevGraph &g, int h, const uint8_t *mask, u64 *deg, hipStream_t s, Scratch &sc,
                           RootClasses &rc) {
    const int32_t n = g.n;
    const int R = h - 1;
    int32_t *cursor = sc.get_n<int32_t>(2 * NBIN);
    u64 *bound = sc.get_n<u64>(1);
    k_enum_init<<<grid_for(n, BLOCK, 4096), BLOCK, 0, s>>>(deg, n, cursor, bound);
    const int blocks = (int)(((int64_t)n + CLASSIFY_TILE - 1) / CLASSIFY_TILE);
    RootOffsets ro{};
    k_classify<false><<<blocks, BLOCK, 0, s>>>(g.row_ptr, g.dag_off, mask, n, R, cursor, nullptr, ro, bound);
    u64 hb = 0;
    Readback(sc).add(rc.hc, cursor, NBIN).add(&hb, bound).run(s);
    if (hb == ~0ull || hb > ~0ull / (u64)h) return false;          // counts could overflow 64 bits
    if (rc.hc[7]) throw Error(-5, "an out-neighbourhood exceeds 2048 vertices (limit of the bitmap kernels, h >= 4)");
    rc.off[0] = 0;
    for (int c = 0; c < NBIN; c++) rc.off[c + 1] = rc.off[c] + rc.hc[c];
    for (int c = 0; c <= NBIN; c++) ro.off[c] = rc.off[c];
    rc.lists = sc.get_n<int32_t>(rc.off[NBIN]);
    k_classify<true><<<blocks, BLOCK, 0, s>>>(g.row_ptr, g.dag_off, mask, n, R, cursor + NBIN, rc.lists, ro, bound);
    return true;
}

bool clique_degrees(const DevGraph &g, int h, const uint8_t *mask, u64 *deg, hipStream_t s, Scratch &sc,
                    KernelTimes *kt, int gs_blocks, EventSpan *span) {
    const int32_t n = g.n;
    if (n == 0) return true;
    if (h == 2) {
        if (mask) k_deg_h2_masked<<<grid_for(n, WAVES_PER_BLOCK, 8192), BLOCK, 0, s>>>(g.row_ptr, g.col, mask, n, deg);
        else k_deg_h2<<<grid_for(n, BLOCK, 8192), BLOCK, 0, s>>>(g.row_ptr, n, deg);
        return true;
    }
    const int R = h - 1;
    RootClasses rc;
    if (!classify_roots(g, h, mask, deg, s, sc, rc)) return false;
    EnumCtx ctx{nullptr, mask, deg};
    EventSpan own, &es = span ? *span : own;
    if (kt) es.begin(s);
    switch (R) {
        case 2: launch_engine<2>(g, ctx, rc.lists, rc.off, rc.hc, s, sc, gs_blocks); break;
        case 3: launch_engine<3>(g, ctx, rc.lists, rc.off, rc.hc, s, sc, gs_blocks); break;
        case 4: launch_engine<4>(g, ctx, rc.lists, rc.off, rc.hc, s, sc, gs_blocks); break;
        case 5: launch_engine<5>(g, ctx, rc.lists, rc.off, rc.hc, s, sc, gs_blocks); break;
        default: throw Error(-1, "h outside [2, 6]");
    }
    if (kt) {
        es.end(s);
        for (int c = 0; c < nclass_of(R); c++) kt->k3_launches += class_roots(R, c, rc.hc) ? 1 : 0;
        if (!span) {
            DSD_HIP(hipStreamSynchronize(s));
            kt->k3_ms += own.ms();
        }
    }
    return true;
}

std::vector<TuneResult> autotune(const DevGraph &g, int h, hipStream_t s, Scratch &sc) {
    std::vector<TuneResult> out;
    if (h < 3 || h > 6) throw Error(-1, "tuning needs h in [3, 6]");
    const int32_t n = g.n;
    if (n == 0) return out;
    const int R = h - 1;
    RootClasses rc;
    u64 *deg = sc.get_n<u64>(n);
    if (!classify_roots(g, h, nullptr, deg, s, sc, rc)) throw Error(-4, "clique counts could exceed 64 bits");
    EnumCtx ctx{nullptr, nullptr, deg};
    DSD_HIP(hipStreamSynchronize(s));
    hipEvent_t e0, e1;
    DSD_HIP(hipEventCreate(&e0));
    DSD_HIP(hipEventCreate(&e1));
    const std::string arch = arch_name();
    for (int c = 0; c < nclass_of(R); c++) {
        const int32_t roots = class_roots(R, c, rc.hc);
        if (!roots) continue;
        // caps in workgroups; the wave class counts four roots a workgroup
        const int per = c == 0 ? WAVES_PER_BLOCK : 1;
        const int need = (int)std::min<int64_t>(((int64_t)roots + per - 1) / per, 1 << 20);
        const bool global = R >= 3 && c >= 3;
        std::vector<int> cands = global ? std::vector<int>{64, 128, 256, 512, 1024}
                                        : std::vector<int>{256, 512, 1024, 2048, 4096, 8192};
        const int def = default_cap(R, c);
        if (std::find(cands.begin(), cands.end(), def) == cands.end()) cands.push_back(def);
        TuneResult tr{c, roots, def, def, 0.0, 0.0};
        std::map<int, double> seen;   // by effective grid
        double best = 1e300;
        for (int cap : cands) {
            const int eff = std::min(cap, need);
            double ms;
            auto it = seen.find(eff);
            if (it != seen.end()) {
                ms = it->second;
            } else {
                ms = 1e300;
                for (int rep = 0; rep < 2; rep++) {   // the faster of two runs
                    DSD_HIP(hipEventRecord(e0, s));
                    launch_one_class(R, c, cap, g, ctx, rc.lists, rc.off, rc.hc, s, sc);
                    DSD_HIP(hipEventRecord(e1, s));
                    DSD_HIP(hipEventSynchronize(e1));
                    float t = 0;
                    DSD_HIP(hipEventElapsedTime(&t, e0, e1));
                    ms = std::min(ms, (double)t);
                }
                seen[eff] = ms;
            }
            if (cap == def) tr.ms_default = ms;
            // a tie keeps the smaller grid (less scratch, fewer idle workgroups)
            if (ms < best * 0.98 || (ms <= best && cap < tr.cap_best)) {
                best = ms;
                tr.cap_best = cap;
            }
        }
        // (a smaller grid within 2 % of the built-in one, but behind it, gives way)
        if (tr.ms_default < best) {
            best = tr.ms_default;
            tr.cap_best = def;
        }
        tr.ms_best = best;
        out.push_back(tr);
        TuneTable &t = tune_table();
        std::lock_guard<std::mutex> lk(t.mu);
        t.env_read = true;
        t.cap[tune_key(arch, h, c)] = tr.cap_best;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    DSD_HIP(hipStreamSynchronize(s));
    return out;
}

void tune_write(const char *path) { tune_save(path); }

}  // namespace dsd
