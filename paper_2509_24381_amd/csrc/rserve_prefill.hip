// Host side of the C ABI declared in include/rserve_prefill.h: argument checks, per-call descriptors and the
// kernel sequence of one decoder layer over one chunk / micro-batch.  All device work goes to the caller's stream.
#include "../../include/rserve_prefill.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "attention.h"
#include "common.h"
#include "elementwise.h"
#include "kv_fp8.h"
#include "kv_transfer.h"
#include "gemm_strip.h"
#include "gemm_skinny.h"
#include "gemm_tile.h"
#include "last_error.h"

namespace {

thread_local std::string g_last_error = "";

void set_last_error(const char* fmt, va_list ap) {
    char buf[512];
    vsnprintf(buf, sizeof(buf), fmt, ap);
    g_last_error = buf;
}

rs_status fail(rs_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    set_last_error(fmt, ap);
    va_end(ap);
    return st;
}

#define RS_HIP(expr)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return fail(RS_EHIP, "%s: %s", #expr, hipGetErrorString(e_));       \
    } while (0)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

constexpr int RING_SLOTS = 32;
constexpr int RING_CHECKPOINT = 8;

// Workspace of rs_prefill_chunk_static.  In host code the array's name is only a handle for hipGetSymbolAddress: each GPU
// holds its own copy at its own address, which static_workspace_lookup fetches once per device (with that device
// current) and every later use goes through.
static __device__ __align__(256) unsigned char g_static_workspace[RS_STATIC_WORKSPACE_BYTES];
constexpr int MAX_DEVICES = 64;
void* g_static_workspace_addr[MAX_DEVICES] = {};   // per device; written under g_static_workspace_mutex
std::mutex g_static_workspace_mutex;

// The address of the current device's copy of the array (the device must be `dev`); looked up on first use.
hipError_t static_workspace_lookup(int dev, void** out) {
    std::lock_guard<std::mutex> lock(g_static_workspace_mutex);
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    if (!g_static_workspace_addr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_workspace));
        if (e != hipSuccess) return e;
        g_static_workspace_addr[dev] = p;
    }
    *out = g_static_workspace_addr[dev];
    return hipSuccess;
}

}  // namespace

rs_status rs_internal_fail(rs_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    set_last_error(fmt, ap);
    va_end(ap);
    return st;
}

struct rs_ctx {
    rs_layer_cfg cfg;
    int qkv_dim, q_dim, kv_dim, group;
    float2* rope_dev = nullptr;  // [max_pos][d/2] (cos, sin)
    // pinned staging ring for per-call descriptors
    char* pinned[RING_SLOTS] = {};
    char* pinned_dev[RING_SLOTS] = {};  // the same buffers as the device addresses them
    // A slot may be overwritten once the first kernel of the call that used it has run.  Recording an event behind that
    // kernel in every call would tell, but an event record holds the stream up for about 6 us; so events are recorded only
    // at checkpoints: after every RING_CHECKPOINT-th use, and - on the stream that is being left - whenever the caller's
    // stream changes.  Uses are numbered; the first checkpoint at or after use u is on u's stream and behind its kernel.
    hipEvent_t slot_done[RING_SLOTS] = {};
    long slot_recorded_at[RING_SLOTS];   // the use number slot_done[slot] was last recorded at (-1: never)
    size_t slot_bytes = 0;
    long use_count = 0;                   // uses so far; use u occupies slot u % RING_SLOTS
    hipStream_t last_stream = nullptr;
    int splitk_override = 0;  // RS_SPLITK environment variable (0 = heuristic)
    int mrope_b0 = 0, mrope_b1 = 0;  // rotary pair j turns with axis 0 below b0, axis 1 below b1, axis 2 above (set in rs_ctx_create)
    bool attn_plain_order = false;  // RS_ATTN_ORDER=plain: attention blocks that share a compute unit stay heaviest-first (no pairing)
    int attn_split = 0;       // RS_ATTN_SPLIT environment variable: parts a block's key range is cut into (0: decided per call)
    int gemm_few = 1;         // RS_NARROW environment variable: 0 keeps every call on the strip GEMMs (no tiles, no few-rows kernel)
    int n_cu = 256;           // compute units of the device: the number of strips a GEMM launch is cut into
    bool has_device = false;  // false: created on a host without a GPU; argument checks work, launches return RS_EHIP
    int device = -1;          // the GPU that was current in rs_ctx_create
    void* static_ws = nullptr;  // that GPU's copy of the static workspace (rs_prefill_chunk_static)
    int lm_rows = 0;          // rows per launch of the first-token head (0: its LDS size not yet set, see rs_lm_head)
    // measurement hook: HIP events around every launch of one step of the layer
    int prof_step = -1;
    int prof_count = 0;
    int prof_every = 1;       // measure every n-th launch of the step
    int prof_seen = 0;        // launches of the step seen since rs_profile_enable
    bool prof_take = false;   // the launch in progress is being measured
    std::vector<hipEvent_t> prof_events;  // (start, stop) pairs
};

// A pool of fixed-size pages in caller-owned device memory.  A page holds 64 tokens of ONE layer: the K tiles [64][d] of
// all KV heads followed by their V^T tiles [d][64].  The free list lives on the host.
struct rs_kv_pool {
    rs_ctx* ctx;
    char* base;
    size_t page_bytes;
    int n_pages;
    bool fp8 = false;              // pages of E4M3 bytes (half the size) for 8-bit caches
    int n_caches = 0;              // paged caches alive on this pool
    std::vector<int> free_pages;   // stack: the back is handed out next
};

struct rs_kv {
    rs_ctx* ctx;
    int n_layers;
    int cap;  // contiguous: capacity in tokens, multiple of 64; paged: unused (see capacity())
    char* base;
    size_t k_bytes;      // one layer's K
    size_t layer_bytes;  // K + V^T
    std::vector<int> len;
    rs_kv_pool* pool = nullptr;             // paged caches only
    std::vector<std::vector<int>> pages;    // paged: pages[layer][block]
    bool fp8 = false;                       // one E4M3 byte per element (contiguous caches only); k_bytes counts bytes
    float k_scale = 1.0f, v_scale = 1.0f;   // 8-bit caches: value = decode(code) * scale
    bool paged() const { return pool != nullptr; }
    uint8_t* kc_of(int layer) const { return reinterpret_cast<uint8_t*>(base + (size_t)layer * layer_bytes); }
    uint8_t* vc_of(int layer) const { return reinterpret_cast<uint8_t*>(base + (size_t)layer * layer_bytes + k_bytes); }
    bf16* k_of(int layer) const { return reinterpret_cast<bf16*>(base + (size_t)layer * layer_bytes); }
    bf16* vt_of(int layer) const { return reinterpret_cast<bf16*>(base + (size_t)layer * layer_bytes + k_bytes); }
    // new pages layer `layer` needs before it can hold n_tokens
    int pages_missing(int layer, long n_tokens) const {
        return paged() ? std::max<long>(0, (n_tokens + 63) / 64 - (long)pages[layer].size()) : 0;
    }
    void take_pages(int layer, long n_tokens) {  // the caller has checked that the pool has enough
        for (int k = pages_missing(layer, n_tokens); k > 0; --k) {
            pages[layer].push_back(pool->free_pages.back());
            pool->free_pages.pop_back();
        }
    }
    void give_back_pages(int layer, long n_tokens) {  // keeps the pages that hold the first n_tokens
        const size_t keep = (size_t)((n_tokens + 63) / 64);
        while (pages[layer].size() > keep) {
            pool->free_pages.push_back(pages[layer].back());
            pages[layer].pop_back();
        }
    }
    // the cache of `layer` as the kernels see it (row0 / T / P left to the caller; `pages` is a device pointer or a marker)
    ReqDesc view(int layer, const int* dev_pages) const {
        ReqDesc d{};
        d.cap = cap;
        d.hkv = ctx->cfg.n_kv_heads;
        if (paged()) {
            d.kcache = reinterpret_cast<bf16*>(pool->base);
            d.pages = dev_pages;
        } else {
            d.kcache = k_of(layer);
            d.vtcache = vt_of(layer);
        }
        return d;
    }
};

namespace {

constexpr int TILE_ROWS = 1024;   // rows of the calls whose projections may run on tiles (choose_route)

struct DescSizes {
    size_t reqs, items, vblocks, rowpos, pagetab, mitems, fp8, total;
    size_t append;   // behind total, in the staging buffer only (KVTails and KVRows)
};

DescSizes desc_sizes(const rs_ctx* c, int max_tokens, int max_requests) {
    DescSizes d;
    const size_t n_items = ((size_t)(max_tokens * (size_t)c->group + 32 * ATT_WAVES_SMALL - 1) / (32 * ATT_WAVES_SMALL) + max_requests) * c->cfg.n_kv_heads +
                           ATT_SPLIT_SLOTS;
    const size_t n_vb = (size_t)max_tokens / 64 + 2 * (size_t)max_requests + 1;
    d.reqs = align_up(sizeof(ReqDesc) * std::max(max_requests, 1), 256);
    d.items = align_up(sizeof(AttnItem) * n_items, 256);
    d.vblocks = align_up(sizeof(KVBlockItem) * n_vb, 256);
    d.rowpos = align_up(3 * sizeof(int) * (size_t)std::max(max_tokens, 1), 256);  // (temporal, height, width) per row
    // block -> page numbers of the paged caches in the call: at most max_pos / 64 + 1 blocks per request
    d.pagetab = align_up(sizeof(int) * (size_t)std::max(max_requests, 1) * ((size_t)c->cfg.max_pos / 64 + 2), 256);
    d.mitems = align_up(sizeof(AttnMergeItem) * ATT_SPLIT_SLOTS, 256);
    d.fp8 = align_up(sizeof(Fp8CacheDesc) * std::max(max_requests, 1), 256);
    d.append = align_up(sizeof(KVTail) * std::max(max_requests, 1) + sizeof(KVRow) * std::min(max_tokens, TILE_ROWS), 256);
    d.total = d.reqs + d.items + d.vblocks + d.rowpos + d.pagetab + d.mitems + d.fp8;
    return d;
}

// Strips per 256-row block of a GEMM with `units` 32-feature units: one workgroup per compute unit when there is enough
// width, never more strips than units, and no more than keep the widest strip as narrow: further ones end no sooner and only
// fetch the token operand once more each (us, strips as many as units of the chip -> this: QKV 2048 rows, 7B, 32 -> 29 strips
// 71.5 -> 69.0, O 32 -> 28: 60.5 -> 58.6; layer call of 512 rows 331 -> 318, gate/up 128 -> 119 strips: 124 -> 118).  Strips of more
// than 5 units are bound by their MFMAs rather than by that fetch: where hardly any has the full width, the others had better end
// sooner (72B, 1200 rows, one strip of 51 with 6 units, the others with 5: down 43 -> 51 strips 503 -> 497; 1700 rows, 4 of 36 with 8:
// O 32 -> 36 strips 209.5 -> 203, down 675 -> 663; but 7B, 1700 rows, O, 4 of 36 with 4 units: 28 strips 52.5, 36 strips 54.9).
int strips_for(const rs_ctx* c, int tiles_m, int splits, int units) {
    const int most = std::max(1, std::min(units, c->n_cu / std::max(1, tiles_m * splits)));
    const int ups = (units + most - 1) / most;
    if (ups > 5 && 6 * (units - most * (ups - 1)) < most) return most;
    return (units + ups - 1) / ups;
}

// Estimated duration (shader clocks) of a residual GEMM cut into `splits` K ranges.  Constants fitted to measurements
// on MI355X: a step of K = 64 costs 256 clocks of matrix-pipe issue per unit plus about 350 of barrier and issue overhead,
// a tile about 20000 for pipeline fill and epilogue, and the reduction kernel moves its bytes at about 2 TB/s.
double gemm_cost_clocks(const rs_ctx* c, int M, int units, int k_steps, int splits) {
    const int tiles_m = (M + GS_BM - 1) / GS_BM;
    const int strips = strips_for(c, tiles_m, splits, units);
    const int waves = (tiles_m * strips * splits + c->n_cu - 1) / c->n_cu;  // rounds of workgroups over the chip
    const int ups = (units + strips - 1) / strips;
    const int ntiles = (ups + GS_MAX_NT - 1) / GS_MAX_NT;
    const double nt = (double)ups / ntiles;
    const int steps = (k_steps + splits - 1) / splits;
    // (a step also moves 32 KB of token fragments per workgroup whatever the tile's width: with three
    // units or fewer that, not the MFMAs, sets its duration - about 1200 clocks measured; without this floor calls of 257
    // to 768 rows kept the O projection unsplit, 3 to 8 us slower than in two or three K ranges)
    const double step = std::max(256.0 * nt + 350.0, 1200.0);
    double clocks = (double)waves * ntiles * (steps * step + 20000.0);
    if (splits > 1) clocks += (double)M * units * 32.0 * (4.0 * splits + 4.0) / 2.0e12 * 1.4e9;
    return clocks;
}

int choose_splitk(const rs_ctx* c, int M, int units, int k_steps) {
    if (c->splitk_override > 0) return std::min(std::min(c->splitk_override, 4), std::max(1, k_steps));  // (the workspace holds 4 planes)
    int best = 1;
    double best_cost = gemm_cost_clocks(c, M, units, k_steps, 1);
    for (int s = 2; s <= 4 && k_steps / s >= 8; ++s) {
        const double cost = gemm_cost_clocks(c, M, units, k_steps, s);
        if (cost < 0.97 * best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

constexpr int MAX_PLANES = 4, MAX_PLANES_FEW = 8, FEW_PLANES_ROWS = 256;   // split-K partial planes: up to 8 in calls of few rows

struct WorkspaceLayout {
    size_t qkv, xf, attn, r, act, partial, attn_split, inv_rms1, inv_rms2, rowss, desc, total;
    int planes;   // that partial has room for
};

WorkspaceLayout ws_layout(const rs_ctx* c, int T, int R) {
    const rs_layer_cfg& f = c->cfg;
    WorkspaceLayout w;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += align_up(bytes, 256);
        return o;
    };
    const size_t t = (size_t)std::max(T, 1);
    const size_t tp = align_up(t, 32);  // fragment-major buffers hold whole blocks of 32 tokens
    w.qkv = take(t * c->qkv_dim * 2);
    w.xf = take(tp * f.hidden * 2);
    w.attn = take(tp * c->q_dim * 2);
    w.r = take(tp * f.hidden * 2);
    w.act = take(tp * f.mlp_inter * 2);
    w.partial = take(MAX_PLANES * t * f.hidden * 4);  // split-K partial planes of [T, H] fp32, and more of them in attn_split, which is free by then
    w.attn_split = take((size_t)ATT_SPLIT_SLOTS * (32 * ATT_WAVES) * (f.head_dim + 2) * 4);  // partial results of split key ranges
    w.planes = T <= FEW_PLANES_ROWS && off - w.partial >= MAX_PLANES_FEW * t * f.hidden * 4 ? MAX_PLANES_FEW : MAX_PLANES;
    w.inv_rms1 = take(tp * 4);
    w.inv_rms2 = take(tp * 4);
    w.rowss = take(tp * (f.hidden / 32) * 4);
    w.desc = take(desc_sizes(c, T, R).total);
    w.total = off;
    return w;
}

// bytes of the bfloat16 copy of an 8-bit cache's first n_tokens (whole 64-token blocks, K and V^T of all KV heads)
size_t fp8_expansion_bytes(const rs_ctx* c, long n_tokens) {
    return (size_t)2 * align_up((size_t)n_tokens, 64) * c->kv_dim * 2;
}

// Weights that one workgroup reads once, and that the L2s (32 MB together) could not keep from one call to the next, are loaded with the
// streaming hint (GS_ONCE): gate/up of 64 rows, 7B (272 MB), 54.2 -> 50.1 us between events, 72B (969 MB) 182 -> 160; smaller ones lose
// by it (tiny layer, gate/up of 200 rows, 1 MB: 9.3 -> 10.1).  In a stack, whose layers together exceed the 256 MB Infinity Cache; one
// layer of hidden 2048 (135 MB) called again and again is still there and loses 3 us (16 rows on 500, 8-bit cache: 73.4 -> 76.6).
constexpr size_t STREAM_BYTES = (size_t)32 << 20;

// Rows up to which the first kernel gives a row a workgroup instead of half a wavefront.
// us per step between events, a workgroup / half a wavefront.  With the sum of planes, hidden 896 at 500 and 600 rows 8.7 / 9.2 and 9.2 /
// 8.9, 2048: 11.6 / 12.0 and 12.6 / 12.1, 3584: 14.1 / 14.5 and 14.4 / 14.3, 5120 at 600 and 700: 19.2 / 19.6 and 21.0 / 20.5, 8192: 26.5 /
// 28.3 and 29.7 / 29.6; without, 3584 at 600: 10.0 / 10.0, 8192 at 500 and 600: 16.4 / 18.0 and 18.7 / 18.0.  The crossing moves from about 530
// rows (narrow layers, or no planes) to 700 (8192 with planes); what one line for all costs is 1.9 us at most (8192, 650 rows).
constexpr int RMS_FEW_ROWS = 608;

// ---- calls of up to TILE_ROWS rows: strips or tiles (gemm_tile.h), and into how many K ranges.
// Estimated ns of a projection: 4.5 us of launch, first loads and epilogue; per step of 64 k the bytes that a workgroup fetches, at the
// rate a compute unit gets them with all of them walking K in step (50 to 60 per ns: the longer K, the less of the token panel an L2
// keeps), or its MFMAs; at least the weights at what HBM streams (6.2 TB/s with the streaming hint, 5.3 without); and the reduction.
// Row blocks of a ragged call count by the average of their live rows.  That is a fit, and ragged launches lie on either side of it: five
// blocks of 64 rows x 128 features, QKV 7B, full (320 rows) 28.8 us, with one row in the last (257) 26.1, which the average puts at 28.0;
// two blocks of 256 and 77 rows on strips, gate/up 7B, 95 to 99, between the average (89) and the fuller block's bytes (104).
// Against measurement (us between events, 3 of them the events'; 7B shape): QKV 250 rows on 64 x 128 27.4 (30.8), 512 on 128 x 96 31
// (35), 1000 on 128 x 160 38.9 (46.8); O 64 rows on 64 x 64 in 4 ranges 14.6 (15.8), 250 on 64 x 64 19.8 (22.0); down 64 rows on
// 64 x 128 in 8 ranges 33 (29.5, its reduction not in it), 250 on 128 x 128 in 4 64 (56.5, likewise).  The estimates rank; they do not predict.
constexpr int TILE_SHAPES = 6;
constexpr int TILE_BLOCKS[TILE_SHAPES] = {2, 2, 4, 4, 4, 4}, TILE_UNITS[TILE_SHAPES] = {2, 4, 2, 3, 4, 5};
double step_ns(double blocks, double units, int steps) {
    const double rate = steps <= 64 ? 60.0 : steps <= 128 ? 54.0 : 50.0;
    return std::max(4096.0 / rate * (blocks + units), 15.3 * blocks * units);
}
double reduce_ns(int M, int units, int splits) { return splits > 1 ? 5500.0 + (double)M * units * 32.0 * (4.0 * splits + 4.0) / 6000.0 : 0.0; }
bool streams_once(int tiles_m, int units, int steps) { return tiles_m == 1 && (size_t)units * steps * 4096 >= STREAM_BYTES; }
double stream_ns(int units, int steps, bool hint) { return 4500.0 + (double)units * steps * 4096.0 / (hint ? 6200.0 : 5300.0); }
double tile_ns(const rs_ctx* c, int shape, int M, int units, int steps, int splits) {
    const int b = TILE_BLOCKS[shape], u = TILE_UNITS[shape];
    const int tiles_m = (M + 32 * b - 1) / (32 * b), wgs = tiles_m * ((units + u - 1) / u) * splits, rounds = (wgs + c->n_cu - 1) / c->n_cu;
    const double fetch = rounds * (4500.0 + (steps + splits - 1) / splits * step_ns((double)((M + 31) / 32) / tiles_m, u, steps));
    return std::max(fetch, stream_ns(units, steps, streams_once(tiles_m, units, steps))) + reduce_ns(M, units, splits);
}
double strip_ns(const rs_ctx* c, int M, int units, int steps, int splits) {
    const int tiles_m = (M + GS_BM - 1) / GS_BM, strips = strips_for(c, tiles_m, splits, units);
    const int rounds = (tiles_m * strips * splits + c->n_cu - 1) / c->n_cu;
    const int ups = (units + strips - 1) / strips, ntiles = (ups + GS_MAX_NT - 1) / GS_MAX_NT;
    const double b = 2.0 * ((M + 63) / 64) / tiles_m;   // (a wavefront without rows loads none)
    const double step = std::max(570.0, step_ns(b, (double)ups / ntiles, steps));   // (its loop takes 1200 clocks with few units)
    const bool hint = splits > 1 && streams_once(tiles_m, units, steps);   // (of the strips compared here launch_gemm gives it to partial sums only)
    return std::max(rounds * (4500.0 + ntiles * ((steps + splits - 1) / splits * step)), stream_ns(units, steps, hint)) + reduce_ns(M, units, splits);
}
struct GemmRoute { int shape, splits; };   // shape -1: strips
// `splits_fixed` > 0: that many K ranges.  `strip_splits`: the K ranges the strips would take.  `most`: the K ranges there are planes for.
// `shapes`: the ones that exist for the epilogue.
GemmRoute choose_route(const rs_ctx* c, int M, int units, int steps, int splits_fixed, int strip_splits, int most, std::initializer_list<int> shapes) {
    GemmRoute best{-1, strip_splits};
    if (!c->gemm_few || M > TILE_ROWS) return best;
    // (a tie goes to the strips, which lose less in a longer call's last block; with one block of rows to the tiles: 72B, 128 rows, down
    // 103.4 -> 97.2, O 44.7 -> 41.3)
    double best_ns = (M <= 128 ? 1.04 : 0.96) * strip_ns(c, M, units, steps, strip_splits);
    for (const int shape : shapes)
        for (int s = splits_fixed > 0 ? splits_fixed : 1; s <= (splits_fixed > 0 ? splits_fixed : most); ++s) {
            if (splits_fixed == 0 && s > 1 && steps / s < 8) break;
            const double ns = tile_ns(c, shape, M, units, steps, s);
            if (ns < best_ns) {
                best_ns = ns;
                best = GemmRoute{shape, s};
            }
        }
    return best;
}

template <int EPI, int BMB, int BU>
rs_status launch_tile_shape(GemmArgs a, int splits, hipStream_t st, int* columns_out) {
    const int units = a.N / 32, steps = a.K / GS_BK;
    a.tiles_m = (a.M + 32 * BMB - 1) / (32 * BMB);
    a.strips = (units + BU - 1) / BU;
    a.steps_per_split = (steps + splits - 1) / splits;
    splits = (steps + a.steps_per_split - 1) / a.steps_per_split;
    if (columns_out) *columns_out = (units + TileShape<BMB, BU>::TN - 1) / TileShape<BMB, BU>::TN;
    const dim3 grid(a.tiles_m * a.strips * splits);
    if (streams_once(a.tiles_m, units, steps)) hipLaunchKernelGGL((gemm_tile_kernel<EPI, BMB, BU, true>), grid, dim3(256), (tile_lds_bytes<BMB, BU>()), st, a);
    else hipLaunchKernelGGL((gemm_tile_kernel<EPI, BMB, BU, false>), grid, dim3(256), (tile_lds_bytes<BMB, BU>()), st, a);
    RS_HIP(hipGetLastError());
    return RS_OK;
}
template <int EPI>
rs_status launch_tile(int shape, const GemmArgs& a, int splits, hipStream_t st, int* columns_out = nullptr) {
    if (shape == 0) return launch_tile_shape<EPI, 2, 2>(a, splits, st, columns_out);
    if (shape == 1) return launch_tile_shape<EPI, 2, 4>(a, splits, st, columns_out);
    if constexpr (EPI == EPI_QKV_ROPE || EPI == EPI_QKV_APPEND) {
        if (shape == 3) return launch_tile_shape<EPI, 4, 3>(a, splits, st, columns_out);
        return launch_tile_shape<EPI, 4, 5>(a, splits, st, columns_out);
    } else {
        if (shape == 2) return launch_tile_shape<EPI, 4, 2>(a, splits, st, columns_out);
        return launch_tile_shape<EPI, 4, 4>(a, splits, st, columns_out);
    }
}
constexpr std::initializer_list<int> QKV_SHAPES = {0, 1, 3, 5}, RESIDUAL_SHAPES = {0, 1, 2, 4};
template <int EPI, int BMB, int BU>
hipError_t allow_tile_lds(hipError_t e) {
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_tile_kernel<EPI, BMB, BU, true>, hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds_bytes<BMB, BU>());
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_tile_kernel<EPI, BMB, BU, false>, hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds_bytes<BMB, BU>());
    return e;
}

// *columns_out (optional) receives the number of strips, i.e. the number of parts the residual epilogue leaves in GemmArgs::rowss.
template <int EPI>
rs_status launch_gemm(const rs_ctx* c, GemmArgs a, int splits, hipStream_t st, int* columns_out = nullptr) {
    a.tiles_m = (a.M + GS_BM - 1) / GS_BM;
    const int units = a.N / 32;
    const int steps = a.K / GS_BK;
    a.steps_per_split = (steps + splits - 1) / splits;
    splits = (steps + a.steps_per_split - 1) / a.steps_per_split;  // no empty K range
    constexpr bool once_epi = EPI == EPI_SWIGLU || EPI == EPI_PARTIAL;
    a.strips = strips_for(c, a.tiles_m, splits, units);
    if (columns_out) *columns_out = a.strips;
    dim3 grid(a.tiles_m * a.strips, splits);
    if (once_epi && streams_once(a.tiles_m, units, steps))
        hipLaunchKernelGGL((gemm_strip_kernel<EPI, once_epi>), grid, dim3(256), GS_LDS_BYTES, st, a);
    else
        hipLaunchKernelGGL(gemm_strip_kernel<EPI>, grid, dim3(256), GS_LDS_BYTES, st, a);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// Which projections of a call of M rows run in gemm_skinny.h.  Its wavefronts each fetch their own copy of the token
// fragments, M K 2 bytes per workgroup: it wins while that is small beside what the strip kernel loses to its ring and its
// reduction.  Measured us per step, strip -> skinny: QKV 7B 1 row 22.0 -> 14.2, 64 rows (M K = 229k) 22.1 -> 18.7, 100 rows
// (358k) 26.2 -> 26.6, 72B 16 rows (131k) 47 -> 42, 64 rows (524k) 54 -> 70;  O 20 rows 19.1 -> 14.9, 64 rows 20.2 -> 18.3 but
// the gate/up kernel then closes 112 parts of its row sums, 2 us;  down 20 rows 37.3 -> 35.6, 64 rows 41 -> 46;  layers as
// narrow as the tiny shape gain up to 128 rows, and in the gate/up projection too (elsewhere that streams 272 MB: 5 TB/s).
// Between the shapes the lines were drawn from, layer call, us, strip kernel only -> these rules, at 32 / 64 / 128 rows on 256 tokens:
// hidden 512 44.6 / 46.2 / 48.4 -> 31.5 / 36.3 / 41.7; 1024 50.2 / 52.8 / 55.1 -> 36.7 / 42.6 / 50.0; 1536 (d 128) 68.3 / 70.5 / 75.8 ->
// 56.8 / 65.1 / 72.0; 2048 67.4 / 69.1 / 74.0 -> 57.9 / 63.3 / 72.2; 72B 32 / 64 / 128 rows 424 / 441 / 475 -> 362 / 390 / 422.
constexpr int SKINNY_ROWS = 128;
bool skinny_qkv(const rs_ctx* c, int M, int K) { return c->gemm_few && M <= SKINNY_ROWS && (long)M * K <= 256 * 1024; }
bool skinny_residual(const rs_ctx* c, int M, int K) { return c->gemm_few && (M <= 32 || (M <= SKINNY_ROWS && K <= 1024)); }
bool skinny_swiglu(const rs_ctx* c, int M, int K) { return c->gemm_few && M <= SKINNY_ROWS && K <= 1024; }

// EPI_QKV_ROPE or EPI_SWIGLU: a wavefront per 32 tokens.
template <int EPI>
rs_status launch_skinny_rows(GemmArgs a, hipStream_t st) {
    a.steps_per_split = a.K / GS_BK;
    const dim3 grid(a.N / 32);
    const int blocks = (a.M + 31) / 32;
    if (blocks == 1) hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 1, 1, 1, 24>), grid, dim3(64), 0, st, a);
    else if (blocks == 2) hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 1, 2, 1, 24>), grid, dim3(128), 0, st, a);
    else hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 1, 4, 1, 16>), grid, dim3(256), 0, st, a);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// A residual projection (EPI_RESIDUAL, one K range) or its partial planes (EPI_PARTIAL).
template <int EPI>
rs_status launch_skinny(const rs_ctx* c, GemmArgs a, int splits, hipStream_t st, int* columns_out = nullptr) {
    const int steps = a.K / GS_BK, units = a.N / 32;
    a.steps_per_split = (steps + splits - 1) / splits;
    splits = (steps + a.steps_per_split - 1) / a.steps_per_split;
    if (columns_out) *columns_out = units;
    const dim3 grid(units, splits);
    const int blocks = (a.M + 31) / 32;
    // eight wavefronts where each still has a few dozen k-steps, four otherwise
    if (blocks > 2) hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 4, 1, 4, 8>), grid, dim3(256), 4 * 4 * 4096, st, a);
    else if (blocks == 2) hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 2, 1, 4, 16>), grid, dim3(256), 4 * 2 * 4096, st, a);
    else if (a.steps_per_split * 4 >= 8 * 32) hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 1, 1, 8, 16>), grid, dim3(512), 8 * 4096, st, a);
    else hipLaunchKernelGGL((gemm_skinny_kernel<EPI, 1, 1, 4, 24>), grid, dim3(256), 4 * 4096, st, a);
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// out = resid + X W^T, through split-K partials when the unsplit launch would leave compute units idle.  X is fragment-
// major; resid and out are row-major or fragment-major as flagged.  When inv_rms_out is given, the RMSNorm factor of the
// next GEMM's input, rsqrt(mean(out[m,:]^2) + eps) per row, is prepared in one of two forms: the split-K reduction writes
// it to inv_rms_out (*rowss_parts_out = 0); an unsplit launch leaves *rowss_parts_out > 0 partial sums of squares per row
// in rowss, which the next GEMM closes itself (GemmArgs::rowss).
// With `defer` (the layers of one rs_prefill_model_batch call) a split-K launch leaves its reduction to the next layer's
// first kernel: *defer then describes the pending sum (splits > 0) and `out` has not been written yet.
struct PendingReduce {
    int splits = 0;             // 0: nothing pending
    const float* partial = nullptr;
    const bf16* resid = nullptr;   // fragment-major
    bf16* out = nullptr;           // row-major
};
rs_status gemm_residual(const rs_ctx* c, const bf16* X, const bf16* W, const bf16* resid, int resid_frag, bf16* out,
                        int out_frag, int M, int N, int K, float* partial, int planes, float* inv_rms_out, float* rowss, int* rowss_parts_out,
                        hipStream_t st, PendingReduce* defer = nullptr) {
    GemmArgs a{};
    a.X = X; a.W = W; a.out = out; a.ldo = N; a.out_frag = out_frag; a.resid = resid; a.ldr = N; a.resid_frag = resid_frag;
    a.partial = partial;
    a.M = M; a.N = N; a.K = K;
    const float eps = c->cfg.rms_eps;
    const bool skinny = skinny_residual(c, M, K);
    int splits = choose_splitk(c, M, N / 32, K / GS_BK);
    int shape = -1;
    if (skinny && c->splitk_override == 0) {   // (a K too long for one compute unit's loads, and units to spare)
        splits = K >= 8192 && 2 * (N / 32) <= c->n_cu ? 2 : 1;
    } else if (!skinny) {
        const GemmRoute route = choose_route(c, M, N / 32, K / GS_BK, c->splitk_override > 0 ? splits : 0, splits, planes, RESIDUAL_SHAPES);
        shape = route.shape;
        splits = route.splits;
    }
    if (splits > 1) {
        const int sps = (K / GS_BK + splits - 1) / splits;
        splits = (K / GS_BK + sps - 1) / sps;
    }
    if (rowss_parts_out) *rowss_parts_out = 0;
    if (splits == 1) {
        a.rowss = inv_rms_out ? rowss : nullptr;
        int* const parts = inv_rms_out ? rowss_parts_out : nullptr;
        if (shape >= 0) return launch_tile<EPI_RESIDUAL>(shape, a, 1, st, parts);
        return skinny ? launch_skinny<EPI_RESIDUAL>(c, a, 1, st, parts) : launch_gemm<EPI_RESIDUAL>(c, a, 1, st, parts);
    }
    rs_status s = shape >= 0 ? launch_tile<EPI_PARTIAL>(shape, a, splits, st)
                : skinny ? launch_skinny<EPI_PARTIAL>(c, a, splits, st) : launch_gemm<EPI_PARTIAL>(c, a, splits, st);
    if (s != RS_OK) return s;
    if (defer && resid_frag && !out_frag && !inv_rms_out) {
        defer->splits = splits; defer->partial = partial; defer->resid = resid; defer->out = out;
        return RS_OK;
    }
    // few rows: a workgroup per row instead of per four
    const auto reduce = [&](auto wpr, auto planes) {
        hipLaunchKernelGGL((splitk_reduce_residual_kernel<decltype(wpr)::value, decltype(planes)::value>), dim3(wpr == 4 ? M : (M + 3) / 4), dim3(256), 0, st,
                           (const float*)partial, splits, resid, N, resid_frag, out, N, out_frag, M, N, inv_rms_out, eps);
    };
    if (splits > MAX_PLANES) reduce(std::integral_constant<int, 4>{}, std::integral_constant<int, MAX_PLANES_FEW>{});
    else if (M <= 512) reduce(std::integral_constant<int, 4>{}, std::integral_constant<int, MAX_PLANES>{});
    else reduce(std::integral_constant<int, 1>{}, std::integral_constant<int, MAX_PLANES>{});
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// Brackets one step of the layer with HIP events on the call's stream when that step is being measured.
struct StepTimer {
    rs_ctx* c;
    hipStream_t st;
    void begin(int step) const {
        if (c->prof_step != step) return;
        c->prof_take = (c->prof_seen++ % c->prof_every == 0) && 2 * (c->prof_count + 1) <= (int)c->prof_events.size();
        if (c->prof_take) (void)hipEventRecord(c->prof_events[2 * c->prof_count], st);
    }
    void end(int step) const {
        if (c->prof_step != step || !c->prof_take) return;
        (void)hipEventRecord(c->prof_events[2 * c->prof_count + 1], st);
        ++c->prof_count;
        c->prof_take = false;
    }
};

template <int D>
rs_status launch_attention_path(const rs_ctx* c, bf16* qkv, bf16* attn, const ReqDesc* d_reqs,
                                const AttnItem* d_items, int n_items, int att_waves, const KVBlockItem* d_vb, int n_vb, bool any_paged,
                                float* split_buf, const AttnMergeItem* d_mitems, int n_mitems, int most_parts, const Fp8CacheDesc* d_fp8, int n_reqs,
                                int n_xblocks, bool append, hipStream_t st, const StepTimer& tm) {
    const rs_layer_cfg& f = c->cfg;
    tm.begin(RS_STEP_APPEND_KV);
    if (d_fp8) {  // 8-bit caches: quantise the new rows into them, then expand what the rows can see for the attention kernel
        hipLaunchKernelGGL(append_kv_fp8_kernel<D>, dim3(n_vb, f.n_kv_heads), dim3(256), 0, st, (const bf16*)qkv, c->qkv_dim,
                           d_reqs, d_fp8, d_vb, f.n_q_heads, f.n_kv_heads);
        RS_HIP(hipGetLastError());
        hipLaunchKernelGGL(kv_expand_fp8_kernel<D>, dim3(n_xblocks, f.n_kv_heads), dim3(256), 0, st, d_reqs, d_fp8, n_reqs);
    } else if (append) {
        hipLaunchKernelGGL(append_kv_kernel<D>, dim3(n_vb, f.n_kv_heads), dim3(256), 0, st, (const bf16*)qkv, c->qkv_dim,
                           d_reqs, d_vb, f.n_q_heads, f.n_kv_heads);
    }
    RS_HIP(hipGetLastError());
    tm.end(RS_STEP_APPEND_KV);
    const float scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)D));
    tm.begin(RS_STEP_ATTENTION);
    const auto attend = [&](auto paged, auto waves) {
        constexpr int W = decltype(waves)::value;
        hipLaunchKernelGGL((attn_prefill_pipelined_kernel<D, decltype(paged)::value, W>), dim3(n_items), dim3(64 * W), 0, st, d_reqs, d_items,
                           (const bf16*)qkv, c->qkv_dim, attn, c->q_dim, c->group, scale_log2e, split_buf);
        const auto merge = [&](auto max_parts, auto early) {
            hipLaunchKernelGGL((attn_merge_kernel<D, W, decltype(max_parts)::value, decltype(early)::value>), dim3(n_mitems, ATT_MERGE_Y), dim3(32 * W), 0, st, d_reqs,
                               d_mitems, (const float*)split_buf, attn, c->q_dim, c->group, scale_log2e);
        };
        if (n_mitems == 0) return;
        if (most_parts <= ATT_FEW_PARTS) merge(std::integral_constant<int, ATT_FEW_PARTS>{}, std::true_type{});
        else if (n_mitems * ATT_MERGE_Y * (W / 2) <= ATT_MERGE_EARLY_WAVES * c->n_cu) merge(std::integral_constant<int, ATT_MAX_PARTS>{}, std::true_type{});
        else merge(std::integral_constant<int, ATT_MAX_PARTS>{}, std::false_type{});
    };
    const auto attend_waves = [&](auto paged) {
        if (att_waves == ATT_WAVES) attend(paged, std::integral_constant<int, ATT_WAVES>{});
        else attend(paged, std::integral_constant<int, ATT_WAVES_SMALL>{});
    };
    if (any_paged) attend_waves(std::true_type{});
    else attend_waves(std::false_type{});
    RS_HIP(hipGetLastError());
    tm.end(RS_STEP_ATTENTION);
    return RS_OK;
}

// Runs an 8-bit cache's export or import kernel over tokens [0, n): in one launch for a contiguous cache, in windows of
// KV_PAGE_WINDOW blocks (whose page numbers ride in the kernel arguments) for a paged one.
template <class Launch>
void for_each_fp8_window(const rs_kv* kv, int layer, int n, Launch&& launch) {
    Fp8CacheDesc fc{};
    fc.hkv = kv->ctx->cfg.n_kv_heads;
    fc.k_scale = kv->k_scale; fc.v_scale = kv->v_scale;
    fc.k_inv = 1.0f / kv->k_scale; fc.v_inv = 1.0f / kv->v_scale;
    KVPageWindow win{};
    if (!kv->paged()) {
        fc.kc = kv->kc_of(layer); fc.vc = kv->vc_of(layer); fc.cap = kv->cap;
        launch(fc, win, 0, 0, n);
        return;
    }
    fc.kc = reinterpret_cast<uint8_t*>(kv->pool->base);
    fc.pages = reinterpret_cast<const int*>(kv->pool->base);   // non-null marker: the numbers come from the window
    const int window_tokens = KV_PAGE_WINDOW * 64;
    for (int t0 = 0; t0 < n; t0 += window_tokens) {
        const int nt = std::min(window_tokens, n - t0);
        const int b0 = t0 / 64, nb = (nt + 63) / 64;
        for (int b = 0; b < nb; ++b) win.page[b] = kv->pages[layer][b0 + b];
        launch(fc, win, b0, t0, nt);
    }
}

// One launch of the export or import kernel over a window's tokens (see kv_transfer.h).
template <class T, class C>
void launch_export(const rs_ctx* c, const ReqDesc& rq, const Fp8CacheDesc& fc, const KVPageWindow& win, int b0, C* k, C* v, int t0, int nt,
                   hipStream_t st) {
    const dim3 grid((nt + 63) / 64, c->cfg.n_kv_heads);
    const int wide = aligned(k, 8 * sizeof(C)) && aligned(v, 8 * sizeof(C));
    if (c->cfg.head_dim == 128) hipLaunchKernelGGL((kv_export_kernel<128, T, C>), grid, dim3(256), 0, st, rq, fc, win, b0, k, v, t0, nt, wide);
    else hipLaunchKernelGGL((kv_export_kernel<64, T, C>), grid, dim3(256), 0, st, rq, fc, win, b0, k, v, t0, nt, wide);
}
template <class T, class C>
void launch_import(const rs_ctx* c, const ReqDesc& rq, const Fp8CacheDesc& fc, const KVPageWindow& win, int b0, const C* k, const C* v, int t0,
                   int nt, hipStream_t st) {
    const dim3 grid((nt + 63) / 64, c->cfg.n_kv_heads);
    const int wide = aligned(k, 8 * sizeof(C)) && aligned(v, 8 * sizeof(C));
    if (c->cfg.head_dim == 128) hipLaunchKernelGGL((kv_import_kernel<128, T, C>), grid, dim3(256), 0, st, rq, fc, win, b0, k, v, t0, nt, wide);
    else hipLaunchKernelGGL((kv_import_kernel<64, T, C>), grid, dim3(256), 0, st, rq, fc, win, b0, k, v, t0, nt, wide);
}

// Tokens [0, len) of an 8-bit cache's layer as bfloat16 values (C = bf16) or as codes (C = uint8_t).
template <class C>
rs_status fp8_export(const rs_kv* kv, int layer, C* k_out, C* v_out, hipStream_t st) {
    for_each_fp8_window(kv, layer, kv->len[layer], [&](const Fp8CacheDesc& fc, const KVPageWindow& win, int b0, int t0, int nt) {
        launch_export<uint8_t>(kv->ctx, ReqDesc{}, fc, win, b0, k_out, v_out, t0, nt, st);
    });
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// Fills tokens [0, n) of an 8-bit cache's layer from bfloat16 values or from codes (the caller has checked n against the
// capacity and, for a paged cache, taken the pages).
template <class C>
rs_status fp8_import(rs_kv* kv, int layer, const C* k_in, const C* v_in, int n, hipStream_t st) {
    for_each_fp8_window(kv, layer, n, [&](const Fp8CacheDesc& fc, const KVPageWindow& win, int b0, int t0, int nt) {
        launch_import<uint8_t>(kv->ctx, ReqDesc{}, fc, win, b0, k_in, v_in, t0, nt, st);
    });
    RS_HIP(hipGetLastError());
    return RS_OK;
}

// The checks rs_kv_import and rs_kv_import_codes share, in the order they are reported; changes nothing.
rs_status import_check(const rs_kv* kv, int layer, int n_tokens) {
    if (layer < 0 || layer >= kv->n_layers) return fail(RS_EINVAL, "layer %d out of range", layer);
    if (n_tokens < 0) return fail(RS_EINVAL, "n_tokens is negative");
    if (!kv->paged() && n_tokens > kv->cap) return fail(RS_ECAPACITY, "%d tokens exceed cache capacity %d", n_tokens, kv->cap);
    if (n_tokens > kv->ctx->cfg.max_pos) return fail(RS_ECAPACITY, "%d tokens exceed max_pos %d", n_tokens, kv->ctx->cfg.max_pos);
    if (kv->paged() && kv->pages_missing(layer, n_tokens) > (int)kv->pool->free_pages.size())
        return fail(RS_ECAPACITY, "the import needs %d new KV pages, the pool has %zu free", kv->pages_missing(layer, n_tokens),
                    kv->pool->free_pages.size());
    return RS_OK;
}

// Runs the export or import kernel over tokens [0, n): in one launch for a contiguous cache, in windows of
// KV_PAGE_WINDOW blocks (whose page numbers ride in the kernel arguments) for a paged one.
template <class Launch>
rs_status for_each_kv_window(const rs_kv* kv, int layer, int n, Launch&& launch) {
    KVPageWindow win{};
    if (!kv->paged()) {
        launch(kv->view(layer, nullptr), win, 0, 0, n);
        return RS_OK;
    }
    const int window_tokens = KV_PAGE_WINDOW * 64;
    for (int t0 = 0; t0 < n; t0 += window_tokens) {
        const int nt = std::min(window_tokens, n - t0);
        const int b0 = t0 / 64, nb = (nt + 63) / 64;
        for (int b = 0; b < nb; ++b) win.page[b] = kv->pages[layer][b0 + b];
        launch(kv->view(layer, reinterpret_cast<const int*>(kv->pool->base)), win, b0, t0, nt);  // non-null marker: paged
    }
    return RS_OK;
}

// pages a call would take from each pool
typedef std::vector<std::pair<rs_kv_pool*, long>> PoolNeed;
void add_need(PoolNeed& need, rs_kv_pool* pool, long n) {
    if (n <= 0) return;
    for (auto& e : need)
        if (e.first == pool) {
            e.second += n;
            return;
        }
    need.emplace_back(pool, n);
}
rs_status check_need(const PoolNeed& need) {
    for (const auto& e : need)
        if (e.second > (long)e.first->free_pages.size())
            return fail(RS_ECAPACITY, "the call needs %ld new KV pages, the pool has %zu free", e.second, e.first->free_pages.size());
    return RS_OK;
}

// Every check of one layer's call; changes nothing.  *total_out receives the number of rows.
rs_status prefill_check(rs_ctx* ctx, const rs_layer_weights* w, int layer, rs_kv* const* kvs, const int* lens, int R,
                        const void* x, void* y, void* ws, size_t ws_bytes, int* total_out, const int* positions3 = nullptr,
                        PoolNeed* pages_needed = nullptr) {
    if (!ctx) return fail(RS_EINVAL, "ctx is null");
    if (!w) return fail(RS_EINVAL, "weights are null");
    const rs_layer_cfg& f = ctx->cfg;
    if (!w->ln1_g || !w->w_qkv || !w->w_o || !w->ln2_g || !w->w_gate_up || !w->w_down)
        return fail(RS_EINVAL, "a weight pointer is null");
    if (f.qkv_bias && !w->b_qkv) return fail(RS_EINVAL, "cfg.qkv_bias is set but b_qkv is null");
    if (R < 0) return fail(RS_EINVAL, "R = %d is negative", R);
    if (R > f.max_requests) return fail(RS_EINVAL, "R = %d exceeds max_requests = %d", R, f.max_requests);
    if (R > 0 && (!kvs || !lens)) return fail(RS_EINVAL, "kvs / chunk_lens is null");
    long total = 0;
    for (int i = 0; i < R; ++i) {
        if (!kvs[i]) return fail(RS_EINVAL, "kvs[%d] is null", i);
        if (kvs[i]->ctx != ctx) return fail(RS_ESTATE, "kvs[%d] belongs to another context", i);
        if (layer < 0 || layer >= kvs[i]->n_layers) return fail(RS_EINVAL, "layer %d out of range for kvs[%d]", layer, i);
        if (lens[i] < 0) return fail(RS_EINVAL, "chunk_lens[%d] = %d is negative", i, lens[i]);
        total += lens[i];
    }
    if (total > f.max_tokens_per_call)
        return fail(RS_EINVAL, "%ld rows exceed max_tokens_per_call = %d", total, f.max_tokens_per_call);
    {
        std::vector<const rs_kv*> sorted(kvs, kvs + R);
        std::sort(sorted.begin(), sorted.end());
        if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end())
            return fail(RS_EINVAL, "the same rs_kv appears twice in one micro-batch");
    }
    for (int i = 1; i < R; ++i)
        if (kvs[i]->fp8 != kvs[0]->fp8)
            return fail(RS_EINVAL, "kvs[%d]: the caches of one call must all be bfloat16 or all be 8-bit", i);
    for (int i = 0; i < R; ++i) {
        const long after = (long)kvs[i]->len[layer] + lens[i];
        if (!kvs[i]->paged() && after > kvs[i]->cap)
            return fail(RS_ECAPACITY, "request %d: %ld tokens exceed cache capacity %d", i, after, kvs[i]->cap);
        if (after > f.max_pos) return fail(RS_ECAPACITY, "request %d: %ld tokens exceed max_pos %d", i, after, f.max_pos);
    }
    if (pages_needed) {  // the caller adds up several layers; one layer's call checks its own need here
        for (int i = 0; i < R; ++i)
            if (kvs[i]->paged()) add_need(*pages_needed, kvs[i]->pool, kvs[i]->pages_missing(layer, (long)kvs[i]->len[layer] + lens[i]));
    } else {
        PoolNeed need;
        for (int i = 0; i < R; ++i)
            if (kvs[i]->paged()) add_need(need, kvs[i]->pool, kvs[i]->pages_missing(layer, (long)kvs[i]->len[layer] + lens[i]));
        const rs_status ps = check_need(need);
        if (ps != RS_OK) return ps;
    }
    *total_out = (int)total;
    if (total == 0) return RS_OK;
    const int T = (int)total;
    if (positions3)
        for (long i = 0; i < 3 * total; ++i)
            if (positions3[i] < 0 || positions3[i] >= f.max_pos)
                return fail(RS_ECAPACITY, "rotary position %d of row %ld is outside [0, max_pos = %d)", positions3[i], i / 3, f.max_pos);
    if (!x || !y) return fail(RS_EINVAL, "x / y is null");
    if (!aligned(x, 16) || !aligned(y, 16)) return fail(RS_EINVAL, "x / y must be 16-byte aligned");
    if (!ws) return fail(RS_EINVAL, "workspace is null");
    if (!aligned(ws, 256)) return fail(RS_EINVAL, "workspace must be 256-byte aligned");
    const WorkspaceLayout L = ws_layout(ctx, T, R);
    size_t expansion = 0;  // 8-bit caches: bfloat16 copies of the blocks the call's rows can see
    for (int i = 0; i < R; ++i)
        if (kvs[i]->fp8 && lens[i] > 0) expansion += fp8_expansion_bytes(ctx, (long)kvs[i]->len[layer] + lens[i]);
    if (ws_bytes < L.total + expansion)
        return fail(RS_EWORKSPACE, "workspace has %zu bytes, this call needs %zu%s", ws_bytes, L.total + expansion,
                    expansion ? " (rs_workspace_bytes_fp8kv: the 8-bit caches are expanded there)" : "");
    // (a caller that adds up the page need of several layers reports that shortage before the missing device)
    if (!pages_needed && !ctx->has_device) return fail(RS_EHIP, "no HIP device: the context was created on a host without a GPU");
    return RS_OK;
}

// Enqueues one layer's call (arguments already checked by prefill_check) and advances the cache lengths.
// `pending_in` (layers after the first of rs_prefill_model_batch): the previous layer's down projection left its split-K
// sum pending; x is then that layer's output buffer, not yet written, and this layer's first kernel produces it.
// `pending_out`: this layer may leave its own down projection pending in the same way (the next layer follows at once).
// `plans`: the attention plan of the call's previous layer, if any; replaced where it does not fit.
rs_status prefill_enqueue(rs_ctx* ctx, const rs_layer_weights* w, int layer, rs_kv* const* kvs, const int* lens, int R, int T,
                          const void* x, void* y, void* ws, void* stream, AttnPlanCache& plans, const int* positions3 = nullptr,
                          const PendingReduce* pending_in = nullptr, PendingReduce* pending_out = nullptr) {
    const rs_layer_cfg& f = ctx->cfg;
    const WorkspaceLayout L = ws_layout(ctx, T, R);
    {   // a call recorded into a HIP graph would replay with stale descriptors: refuse it, before anything changes
        hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(reinterpret_cast<hipStream_t>(stream), &capturing) != hipSuccess) (void)hipGetLastError();
        else if (capturing != hipStreamCaptureStatusNone) return fail(RS_ESTATE, "the stream is capturing a HIP graph");
    }

    // Pages taken below go back to their pools if a later host-side check refuses the call (nothing may change on a
    // status other than RS_OK); from the first launch on they stay.
    struct PageRollback {
        struct Entry { rs_kv* kv; int layer; int len; };
        std::vector<Entry> taken;
        bool armed = true;
        ~PageRollback() {
            if (!armed) return;
            for (auto it = taken.rbegin(); it != taken.rend(); ++it) it->kv->give_back_pages(it->layer, it->len);
        }
    } rollback;

    // ---- host descriptors
    std::vector<ReqDesc> reqs;
    std::vector<KVBlockItem> vbs;
    std::vector<int> rowpos;
    std::vector<int> pagetab;
    std::vector<Fp8CacheDesc> fp8s;
    int n_xblocks = 0;
    size_t expansion_off = L.total;
    rowpos.reserve(3 * (size_t)T);
    const DescSizes ds = desc_sizes(ctx, T, R);
    char* wsb = reinterpret_cast<char*>(ws);
    const int* d_pagetab = reinterpret_cast<const int*>(wsb + L.desc + ds.reqs + ds.items + ds.vblocks + ds.rowpos);
    std::vector<AttnRequest> att_reqs;
    // calls of few rows on bfloat16 caches: k and v go straight from the QKV projection into them
    const bool qkv_few = skinny_qkv(ctx, T, f.hidden);
    const int qkv_shape = qkv_few ? -1 : choose_route(ctx, T, ctx->qkv_dim / 32, f.hidden / GS_BK, 1, 1, 1, QKV_SHAPES).shape;
    const bool fused_append = T <= TILE_ROWS && (qkv_few || qkv_shape >= 0) && !kvs[0]->fp8;
    std::vector<KVTail> tails;
    std::vector<KVRow> kv_places;
    if (fused_append) kv_places.reserve(T);
    int row0 = 0;
    for (int i = 0; i < R; ++i) {
        const int Ti = lens[i];
        if (Ti == 0) continue;
        rs_kv* kv = kvs[i];
        const int P = kv->len[layer];
        if (kv->paged() && kv->pages_missing(layer, (long)P + Ti) > 0) rollback.taken.push_back({kv, layer, P});
        kv->take_pages(layer, (long)P + Ti);   // (paged caches; prefill_check has made sure the pool has them)
        ReqDesc d = kv->view(layer, d_pagetab + pagetab.size());
        d.row0 = row0; d.T = Ti; d.P = P;
        if (kv->fp8) {  // the kernels append to the 8-bit cache and attend to its expansion in the workspace
            Fp8CacheDesc fc{};
            if (kv->paged()) {   // the 8-bit kernels look the pages up; attention reads the (contiguous) expansion
                fc.kc = reinterpret_cast<uint8_t*>(kv->pool->base);
                fc.pages = d.pages;
                d.pages = nullptr;
            } else {
                fc.kc = kv->kc_of(layer); fc.vc = kv->vc_of(layer); fc.cap = kv->cap;
            }
            fc.xb0 = n_xblocks; fc.hkv = f.n_kv_heads;
            fc.k_scale = kv->k_scale; fc.v_scale = kv->v_scale;
            fc.k_inv = 1.0f / kv->k_scale; fc.v_inv = 1.0f / kv->v_scale;
            fp8s.push_back(fc);
            const size_t plane = fp8_expansion_bytes(ctx, (long)P + Ti) / 2;
            d.kcache = reinterpret_cast<bf16*>(wsb + expansion_off);
            d.vtcache = reinterpret_cast<bf16*>(wsb + expansion_off + plane);
            d.cap = (int)align_up((size_t)P + Ti, 64);
            expansion_off += 2 * plane;
            n_xblocks += d.cap / 64;
        }
        if (kv->paged()) pagetab.insert(pagetab.end(), kv->pages[layer].begin(), kv->pages[layer].end());
        const int ri = (int)reqs.size();
        reqs.push_back(d);
        att_reqs.push_back(AttnRequest{Ti, P});
        if (fused_append) {
            const size_t tile = (size_t)64 * f.head_dim * 2, head = kv->paged() ? tile : (size_t)kv->cap * f.head_dim * 2;
            KVRow at{};
            at.head_bytes = head;
            for (int p = P; p < P + Ti; ++p) {
                if (p == P || p % 64 == 0) {   // the tiles of token p's block, KV head 0
                    if (kv->paged()) {
                        at.k = (uint64_t)(uintptr_t)kv->pool->base + (size_t)kv->pages[layer][p / 64] * kv->pool->page_bytes;
                        at.v = at.k + (size_t)f.n_kv_heads * tile;
                    } else {
                        at.k = (uint64_t)(uintptr_t)kv->k_of(layer) + (size_t)(p / 64) * tile;
                        at.v = (uint64_t)(uintptr_t)kv->vt_of(layer) + (size_t)(p / 64) * tile;
                    }
                }
                kv_places.push_back(KVRow{at.k + (size_t)(p % 64) * f.head_dim * 2, at.v + (size_t)(p % 64) * 2, head});
            }
            tails.push_back(KVTail{at.v, head, (P + Ti - 1) % 64 + 1, 0});
        }
        for (int b = P / 64; b <= (P + Ti - 1) / 64; ++b) vbs.push_back(KVBlockItem{ri, b});
        for (int t = 0; t < Ti; ++t)
            for (int ax = 0; ax < 3; ++ax) rowpos.push_back(positions3 ? positions3[3 * (size_t)(row0 + t) + ax] : P + t);
        row0 += Ti;
    }
    if (plans.reqs != att_reqs) {
        plans.plan = plan_attention(AttnPlanSettings{ctx->n_cu, ctx->attn_split, ctx->attn_plain_order}, att_reqs, ctx->group, f.n_kv_heads);
        plans.reqs.swap(att_reqs);
    }
    const AttnPlan& plan = plans.plan;
    const std::vector<AttnItem>& items = plan.items;
    const std::vector<AttnMergeItem>& mitems = plan.merges;

    if (sizeof(ReqDesc) * reqs.size() > ds.reqs || sizeof(AttnItem) * items.size() > ds.items ||
        sizeof(KVBlockItem) * vbs.size() > ds.vblocks || sizeof(int) * rowpos.size() > ds.rowpos ||
        sizeof(int) * pagetab.size() > ds.pagetab || sizeof(AttnMergeItem) * mitems.size() > ds.mitems ||
        sizeof(Fp8CacheDesc) * fp8s.size() > ds.fp8 || (!fp8s.empty() && fp8s.size() != reqs.size()) ||
        sizeof(KVTail) * tails.size() + sizeof(KVRow) * kv_places.size() > ds.append || ds.total + ds.append > ctx->slot_bytes)
        return fail(RS_EINVAL, "internal: descriptor sizing");

    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const long use = ctx->use_count;
    const int slot = (int)(use % RING_SLOTS);
    if (use > 0 && st != ctx->last_stream) {  // leaving a stream: a checkpoint behind its last use, unless there is one
        const int prev = (int)((use - 1) % RING_SLOTS);
        if (ctx->slot_recorded_at[prev] != use - 1) {
            if (hipEventRecord(ctx->slot_done[prev], ctx->last_stream) != hipSuccess) {
                (void)hipGetLastError();       // (the stream is gone: wait for everything instead)
                RS_HIP(hipDeviceSynchronize());
                RS_HIP(hipEventRecord(ctx->slot_done[prev], st));
            }
            ctx->slot_recorded_at[prev] = use - 1;
        }
    }
    if (use >= RING_SLOTS) {  // the slot's previous use: wait for the first checkpoint at or after it
        const long old = use - RING_SLOTS;
        bool waited = false;
        for (long u = old; u < old + RING_CHECKPOINT && !waited; ++u)
            if (ctx->slot_recorded_at[u % RING_SLOTS] == u) {
                RS_HIP(hipEventSynchronize(ctx->slot_done[u % RING_SLOTS]));
                waited = true;
            }
        if (!waited) return fail(RS_EINVAL, "internal: no checkpoint behind use %ld of the descriptor ring", old);
    }
    char* stage = ctx->pinned[slot];
    memcpy(stage, reqs.data(), sizeof(ReqDesc) * reqs.size());
    memcpy(stage + ds.reqs, items.data(), sizeof(AttnItem) * items.size());
    memcpy(stage + ds.reqs + ds.items, vbs.data(), sizeof(KVBlockItem) * vbs.size());
    memcpy(stage + ds.reqs + ds.items + ds.vblocks, rowpos.data(), sizeof(int) * rowpos.size());
    memcpy(stage + ds.reqs + ds.items + ds.vblocks + ds.rowpos, pagetab.data(), sizeof(int) * pagetab.size());
    memcpy(stage + ds.reqs + ds.items + ds.vblocks + ds.rowpos + ds.pagetab, mitems.data(), sizeof(AttnMergeItem) * mitems.size());
    memcpy(stage + ds.reqs + ds.items + ds.vblocks + ds.rowpos + ds.pagetab + ds.mitems, fp8s.data(), sizeof(Fp8CacheDesc) * fp8s.size());
    // (behind the descriptors; the first kernel copies them to where the SwiGLU output will be, which is free until then)
    const size_t append_bytes = fused_append ? align_up(sizeof(KVTail) * tails.size() + sizeof(KVRow) * kv_places.size(), 16) : 0;
    memcpy(stage + ds.total, tails.data(), sizeof(KVTail) * tails.size());
    memcpy(stage + ds.total + sizeof(KVTail) * tails.size(), kv_places.data(), sizeof(KVRow) * kv_places.size());
    const KVRow* const kv_rows = fused_append ? reinterpret_cast<const KVRow*>(wsb + L.act + sizeof(KVTail) * tails.size()) : nullptr;
    // (the first kernel below copies the staged descriptors into the workspace; the slot is free again once it has run)
    const ReqDesc* d_reqs = reinterpret_cast<const ReqDesc*>(wsb + L.desc);
    const AttnItem* d_items = reinterpret_cast<const AttnItem*>(wsb + L.desc + ds.reqs);
    const KVBlockItem* d_vb = reinterpret_cast<const KVBlockItem*>(wsb + L.desc + ds.reqs + ds.items);
    const int* d_rowpos = reinterpret_cast<const int*>(wsb + L.desc + ds.reqs + ds.items + ds.vblocks);
    const AttnMergeItem* d_mitems =
        reinterpret_cast<const AttnMergeItem*>(wsb + L.desc + ds.reqs + ds.items + ds.vblocks + ds.rowpos + ds.pagetab);
    float* attn_split = reinterpret_cast<float*>(wsb + L.attn_split);
    const Fp8CacheDesc* d_fp8 = fp8s.empty() ? nullptr :
        reinterpret_cast<const Fp8CacheDesc*>(wsb + L.desc + ds.reqs + ds.items + ds.vblocks + ds.rowpos + ds.pagetab + ds.mitems);

    bf16* qkv = reinterpret_cast<bf16*>(wsb + L.qkv);
    bf16* xf = reinterpret_cast<bf16*>(wsb + L.xf);
    bf16* attn = reinterpret_cast<bf16*>(wsb + L.attn);
    bf16* r = reinterpret_cast<bf16*>(wsb + L.r);
    bf16* act = reinterpret_cast<bf16*>(wsb + L.act);
    float* partial = reinterpret_cast<float*>(wsb + L.partial);
    float* inv_rms1 = reinterpret_cast<float*>(wsb + L.inv_rms1);
    float* inv_rms2 = reinterpret_cast<float*>(wsb + L.inv_rms2);
    float* rowss = reinterpret_cast<float*>(wsb + L.rowss);
    const bf16* xb = reinterpret_cast<const bf16*>(x);
    bf16* yb = reinterpret_cast<bf16*>(y);
    const int H = f.hidden, I = f.mlp_inter;
    rs_status s;
    const StepTimer tm{ctx, st};

    rollback.armed = false;   // every host-side check has passed: from here on the call is launched
    // 1/rms of every input row (the first RMSNorm; its gain lives in the packed W_qkv)
    tm.begin(RS_STEP_ROW_RMS);
    // and, in the same pass, x in the GEMMs' fragment-major token-operand layout
    const int desc_chunks = (int)(ds.total / 16);
    // (the pending sum reads the previous layer's r and partial planes, which this layer overwrites only later)
    const bool pending = pending_in && pending_in->splits > 0;
    const ReduceSource red = pending ? ReduceSource{pending_in->partial, pending_in->splits, pending_in->resid, pending_in->out} : ReduceSource{};
    const AppendPrep app{reinterpret_cast<uint4*>(wsb + L.act), (int)(append_bytes / 16), (int)tails.size(), f.n_kv_heads, f.head_dim, tails.empty() ? KVTail{} : tails[0]};
    const auto first_kernel = [&](auto planes, auto lanes) {
        constexpr int LANES = decltype(lanes)::value;
        hipLaunchKernelGGL((rms_and_fragment_major_kernel<decltype(planes)::value, LANES>),
                           dim3((LANES == 256 ? T : (T + RMS_ROWS - 1) / RMS_ROWS) + (desc_chunks + app.chunks + 255) / 256 + app.tails * app.hkv), dim3(256),
                           0, st, xb, xf, inv_rms1, T, H, f.rms_eps, reinterpret_cast<const uint4*>(ctx->pinned_dev[slot]),
                           reinterpret_cast<uint4*>(wsb + L.desc), desc_chunks, red, app);
    };
    static_assert(FEW_PLANES_ROWS <= RMS_FEW_ROWS, "more than MAX_PLANES planes: a workgroup per row");
    const auto first_kernel_lanes = [&](auto planes) {
        if (T <= RMS_FEW_ROWS) first_kernel(planes, std::integral_constant<int, 256>{});
        else first_kernel(planes, std::integral_constant<int, 32>{});
    };
    if (!pending) first_kernel_lanes(std::integral_constant<int, 0>{});
    else if (red.splits > MAX_PLANES) first_kernel(std::integral_constant<int, MAX_PLANES_FEW>{}, std::integral_constant<int, 256>{});
    else first_kernel_lanes(std::integral_constant<int, MAX_PLANES>{});
    RS_HIP(hipGetLastError());
    if (use % RING_CHECKPOINT == RING_CHECKPOINT - 1) {
        RS_HIP(hipEventRecord(ctx->slot_done[slot], st));
        ctx->slot_recorded_at[slot] = use;
    } else {
        ctx->slot_recorded_at[slot] = -1;   // (what was recorded here belonged to the slot's previous use)
    }
    ctx->last_stream = st;
    ctx->use_count = use + 1;
    tm.end(RS_STEP_ROW_RMS);
    // qkv = rope( (x Wqkv'^T) / rms + b )
    tm.begin(RS_STEP_QKV_GEMM);
    {
        GemmArgs a{};
        a.X = xf; a.W = (const bf16*)w->w_qkv; a.out = qkv; a.ldo = ctx->qkv_dim;
        a.bias = f.qkv_bias ? (const bf16*)w->b_qkv : nullptr;
        a.row_scale = inv_rms1; a.row_pos = d_rowpos; a.rope_cs = (const float2*)ctx->rope_dev;
        a.rope_cols = ctx->q_dim + ctx->kv_dim; a.head_dim = f.head_dim;
        a.mrope_b0 = ctx->mrope_b0; a.mrope_b1 = ctx->mrope_b1;
        a.M = T; a.N = ctx->qkv_dim; a.K = H;
        a.kv_rows = kv_rows; a.q_cols = ctx->q_dim;
        if (fused_append) s = qkv_few ? launch_skinny_rows<EPI_QKV_APPEND>(a, st) : launch_tile<EPI_QKV_APPEND>(qkv_shape, a, 1, st);
        else if (qkv_few) s = launch_skinny_rows<EPI_QKV_ROPE>(a, st);
        else s = qkv_shape >= 0 ? launch_tile<EPI_QKV_ROPE>(qkv_shape, a, 1, st) : launch_gemm<EPI_QKV_ROPE>(ctx, a, 1, st);
        if (s != RS_OK) return s;
    }
    tm.end(RS_STEP_QKV_GEMM);
    int most_parts = 0;
    for (const AttnMergeItem& item : mitems) most_parts = std::max(most_parts, item.n_parts);
    // cache append, attention
    if (f.head_dim == 128)
        s = launch_attention_path<128>(ctx, qkv, attn, d_reqs, d_items, (int)items.size(), plan.waves, d_vb, (int)vbs.size(), !pagetab.empty() && fp8s.empty(),
                                       attn_split, d_mitems, (int)mitems.size(), most_parts, d_fp8, (int)reqs.size(), n_xblocks, kv_rows == nullptr, st, tm);
    else
        s = launch_attention_path<64>(ctx, qkv, attn, d_reqs, d_items, (int)items.size(), plan.waves, d_vb, (int)vbs.size(), !pagetab.empty() && fp8s.empty(),
                                      attn_split, d_mitems, (int)mitems.size(), most_parts, d_fp8, (int)reqs.size(), n_xblocks, kv_rows == nullptr, st, tm);
    if (s != RS_OK) return s;
    // r = x + attn Wo^T, and 1/rms of every row of r (the second RMSNorm; its gain lives in the packed W_gate_up)
    tm.begin(RS_STEP_O_GEMM);
    int rowss_parts = 0;
    if ((s = gemm_residual(ctx, attn, (const bf16*)w->w_o, xb, 0, r, 1, T, H, ctx->q_dim, partial, L.planes, inv_rms2, rowss, &rowss_parts, st)) != RS_OK) return s;
    tm.end(RS_STEP_O_GEMM);
    // act = silu((r Wg'^T) / rms) * ((r Wu'^T) / rms)
    tm.begin(RS_STEP_GATE_UP_GEMM);
    {
        GemmArgs a{};
        a.X = r; a.W = (const bf16*)w->w_gate_up; a.out = act; a.ldo = I; a.out_frag = 1;
        a.row_scale = inv_rms2;
        if (rowss_parts > 0) {   // the output projection ran unsplit: its per-column sums of squares, closed in this kernel
            a.rowss = rowss; a.rowss_parts = rowss_parts; a.rms_eps = f.rms_eps;
        }
        a.M = T; a.N = 2 * I; a.K = H;
        if ((s = skinny_swiglu(ctx, T, H) ? launch_skinny_rows<EPI_SWIGLU>(a, st) : launch_gemm<EPI_SWIGLU>(ctx, a, 1, st)) != RS_OK) return s;
    }
    tm.end(RS_STEP_GATE_UP_GEMM);
    // y = r + act Wd^T
    tm.begin(RS_STEP_DOWN_GEMM);
    if ((s = gemm_residual(ctx, act, (const bf16*)w->w_down, r, 1, yb, 0, T, H, I, partial, L.planes, nullptr, nullptr, nullptr, st, pending_out)) != RS_OK) return s;
    tm.end(RS_STEP_DOWN_GEMM);

    for (int i = 0; i < R; ++i) kvs[i]->len[layer] += lens[i];
    return RS_OK;
}

rs_status prefill_impl(rs_ctx* ctx, const rs_layer_weights* w, int layer, rs_kv* const* kvs, const int* lens, int R,
                       const void* x, void* y, void* ws, size_t ws_bytes, void* stream, const int* positions3 = nullptr) {
    int T = 0;
    const rs_status s = prefill_check(ctx, w, layer, kvs, lens, R, x, y, ws, ws_bytes, &T, positions3);
    if (s != RS_OK || T == 0) return s;
    AttnPlanCache plans;
    return prefill_enqueue(ctx, w, layer, kvs, lens, R, T, x, y, ws, stream, plans, positions3);
}

}  // namespace

// =============================================================================================== C ABI
extern "C" {

const char* rs_last_error(void) { return g_last_error.c_str(); }
int rs_version(void) { return 1; }

rs_status rs_ctx_create(const rs_layer_cfg* cfg, rs_ctx** out) {
    if (!cfg || !out) return fail(RS_EINVAL, "cfg / out is null");
    *out = nullptr;
    const rs_layer_cfg& f = *cfg;
    if (f.hidden <= 0 || f.n_q_heads <= 0 || f.n_kv_heads <= 0 || f.mlp_inter <= 0 || f.max_tokens_per_call <= 0 ||
        f.max_requests <= 0 || f.max_pos <= 0)
        return fail(RS_EINVAL, "sizes must be positive");
    if (f.head_dim != 64 && f.head_dim != 128) return fail(RS_EINVAL, "head_dim must be 64 or 128");
    if (f.n_q_heads % f.n_kv_heads) return fail(RS_EINVAL, "n_kv_heads must divide n_q_heads");
    const int q_dim = f.n_q_heads * f.head_dim, kv_dim = f.n_kv_heads * f.head_dim, qkv_dim = q_dim + 2 * kv_dim;
    if (f.hidden % 64) return fail(RS_EINVAL, "hidden must be a multiple of 64");
    if (f.mlp_inter % 64) return fail(RS_EINVAL, "mlp_inter must be a multiple of 64");
    if (!(f.rms_eps >= 0.0f) || !(f.rope_theta > 0.0f)) return fail(RS_EINVAL, "rms_eps / rope_theta out of range");
    if ((size_t)f.max_tokens_per_call * (size_t)std::max(qkv_dim, f.mlp_inter) * 2 >= (size_t)1 << 31)
        return fail(RS_EINVAL, "max_tokens_per_call too large for 32-bit row offsets");
    if ((size_t)f.max_tokens_per_call * (size_t)f.hidden * 4 >= (size_t)1 << 31)
        return fail(RS_EINVAL, "max_tokens_per_call * hidden too large for 32-bit offsets into a split-K plane");
    if ((size_t)std::max(2 * f.mlp_inter, qkv_dim) * (size_t)f.hidden * 2 >= (size_t)1 << 31 ||
        (size_t)f.hidden * (size_t)f.mlp_inter * 2 >= (size_t)1 << 31)
        return fail(RS_EINVAL, "weight matrix too large for 32-bit row offsets");

    rs_ctx* c = new rs_ctx();
    c->cfg = f;
    c->q_dim = q_dim; c->kv_dim = kv_dim; c->qkv_dim = qkv_dim; c->group = f.n_q_heads / f.n_kv_heads;
    c->mrope_b0 = c->mrope_b1 = f.head_dim / 2;  // 1-D RoPE: every pair turns with the first axis
    if (const char* e = getenv("RS_SPLITK")) c->splitk_override = atoi(e);
    if (const char* e = getenv("RS_NARROW")) c->gemm_few = atoi(e);
    if (const char* e = getenv("RS_ATTN_ORDER")) c->attn_plain_order = strcmp(e, "plain") == 0;
    if (const char* e = getenv("RS_ATTN_SPLIT")) c->attn_split = std::max(0, std::min(atoi(e), ATT_MAX_PARTS));
    auto cleanup = [&](rs_status s) { rs_ctx_destroy(c); return s; };

    c->slot_bytes = desc_sizes(c, f.max_tokens_per_call, f.max_requests).total + desc_sizes(c, f.max_tokens_per_call, f.max_requests).append;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess || n_dev <= 0) {
        (void)hipGetLastError();
        *out = c;  // host-only context: every check that precedes a launch still works
        return RS_OK;
    }
    c->has_device = true;

    // RoPE table from fp64 angles
    const int half = f.head_dim / 2;
    std::vector<float2> table((size_t)f.max_pos * half);
    std::vector<double> inv_freq(half);
    for (int j = 0; j < half; ++j) inv_freq[j] = std::pow((double)f.rope_theta, -2.0 * j / f.head_dim);
    for (int p = 0; p < f.max_pos; ++p)
        for (int j = 0; j < half; ++j) {
            const double ang = (double)p * inv_freq[j];
            table[(size_t)p * half + j] = make_float2((float)std::cos(ang), (float)std::sin(ang));
        }
    hipError_t e = hipMalloc((void**)&c->rope_dev, table.size() * sizeof(float2));
    if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipMalloc(rope table): %s", hipGetErrorString(e)));
    e = hipMemcpy(c->rope_dev, table.data(), table.size() * sizeof(float2), hipMemcpyHostToDevice);
    if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipMemcpy(rope table): %s", hipGetErrorString(e)));

    for (int i = 0; i < RING_SLOTS; ++i) {
        e = hipHostMalloc((void**)&c->pinned[i], c->slot_bytes, hipHostMallocDefault);
        if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipHostMalloc: %s", hipGetErrorString(e)));
        e = hipHostGetDevicePointer((void**)&c->pinned_dev[i], c->pinned[i], 0);
        if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipHostGetDevicePointer: %s", hipGetErrorString(e)));
        e = hipEventCreateWithFlags(&c->slot_done[i], hipEventDisableTiming);
        if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipEventCreate: %s", hipGetErrorString(e)));
        c->slot_recorded_at[i] = -1;
    }
    int dev = 0, n_cu = 0;
    e = hipGetDevice(&dev);
    if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipGetDevice: %s", hipGetErrorString(e)));
    c->device = dev;
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n_cu > 0) c->n_cu = n_cu;
    e = static_workspace_lookup(dev, &c->static_ws);
    if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipGetSymbolAddress(static workspace): %s", hipGetErrorString(e)));
    if (const char* e = getenv("RS_NCU")) {  // test hook: fewer, wider strips exercise every tile width on small shapes
        if (atoi(e) > 0) c->n_cu = atoi(e);
    }
    // kernels that use more than 64 KB of LDS must opt in
    e = hipFuncSetAttribute((const void*)gemm_strip_kernel<EPI_QKV_ROPE>, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS_BYTES);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_strip_kernel<EPI_RESIDUAL>, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS_BYTES);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_strip_kernel<EPI_SWIGLU>, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS_BYTES);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_strip_kernel<EPI_PARTIAL>, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS_BYTES);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_strip_kernel<EPI_SWIGLU, true>, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS_BYTES);
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)gemm_strip_kernel<EPI_PARTIAL, true>, hipFuncAttributeMaxDynamicSharedMemorySize, GS_LDS_BYTES);
    e = allow_tile_lds<EPI_QKV_ROPE, 4, 5>(allow_tile_lds<EPI_QKV_ROPE, 4, 3>(allow_tile_lds<EPI_QKV_ROPE, 2, 4>(allow_tile_lds<EPI_QKV_ROPE, 2, 2>(e))));
    e = allow_tile_lds<EPI_QKV_APPEND, 4, 5>(allow_tile_lds<EPI_QKV_APPEND, 4, 3>(allow_tile_lds<EPI_QKV_APPEND, 2, 4>(allow_tile_lds<EPI_QKV_APPEND, 2, 2>(e))));
    e = allow_tile_lds<EPI_RESIDUAL, 4, 4>(allow_tile_lds<EPI_RESIDUAL, 4, 2>(allow_tile_lds<EPI_RESIDUAL, 2, 4>(allow_tile_lds<EPI_RESIDUAL, 2, 2>(e))));
    e = allow_tile_lds<EPI_PARTIAL, 4, 4>(allow_tile_lds<EPI_PARTIAL, 4, 2>(allow_tile_lds<EPI_PARTIAL, 2, 4>(allow_tile_lds<EPI_PARTIAL, 2, 2>(e))));
    if (e != hipSuccess) return cleanup(fail(RS_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e)));
    *out = c;
    return RS_OK;
}

void rs_ctx_destroy(rs_ctx* c) {
    if (!c) return;
    for (hipEvent_t e : c->prof_events) (void)hipEventDestroy(e);
    if (c->rope_dev) (void)hipFree(c->rope_dev);
    for (int i = 0; i < RING_SLOTS; ++i) {
        if (c->slot_done[i]) (void)hipEventDestroy(c->slot_done[i]);
        if (c->pinned[i]) (void)hipHostFree(c->pinned[i]);
    }
    delete c;
}

size_t rs_weights_packed_bytes(const rs_ctx* c) {
    if (!c) return 0;
    const rs_layer_cfg& f = c->cfg;
    const size_t H = f.hidden, I = f.mlp_inter;
    size_t b = 0;
    b += align_up(H * 2, 256) * 2;                    // gains
    b += align_up((size_t)c->qkv_dim * H * 2, 256);   // w_qkv
    b += align_up((size_t)c->qkv_dim * 2, 256);       // b_qkv
    b += align_up(H * c->q_dim * 2, 256);             // w_o
    b += align_up(2 * I * H * 2, 256);                // w_gate_up
    b += align_up(H * I * 2, 256);                    // w_down
    return b;
}

rs_status rs_weights_pack(rs_ctx* c, const rs_layer_weights* src, void* dst, size_t dst_bytes, rs_layer_weights* packed,
                          void* stream) {
    if (!c || !src || !dst || !packed) return fail(RS_EINVAL, "null argument");
    const rs_layer_cfg& f = c->cfg;
    if (!src->ln1_g || !src->w_qkv || !src->w_o || !src->ln2_g || !src->w_gate_up || !src->w_down)
        return fail(RS_EINVAL, "a source weight pointer is null");
    if (f.qkv_bias && !src->b_qkv) return fail(RS_EINVAL, "cfg.qkv_bias is set but b_qkv is null");
    if (!aligned(dst, 256)) return fail(RS_EINVAL, "dst must be 256-byte aligned");
    if (!aligned(src->w_gate_up, 16) || !aligned(src->w_qkv, 16) || !aligned(src->ln1_g, 16) || !aligned(src->ln2_g, 16))
        return fail(RS_EINVAL, "source weights must be 16-byte aligned");
    if (dst_bytes < rs_weights_packed_bytes(c)) return fail(RS_EWORKSPACE, "dst has %zu bytes, need %zu", dst_bytes, rs_weights_packed_bytes(c));
    if (!c->has_device) return fail(RS_EHIP, "no HIP device");
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const size_t H = f.hidden, I = f.mlp_inter;
    char* p = reinterpret_cast<char*>(dst);
    auto copy = [&](const void* s, size_t bytes, const void** slot) -> hipError_t {
        *slot = p;
        hipError_t e = hipMemcpyAsync(p, s, bytes, hipMemcpyDeviceToDevice, st);
        p += align_up(bytes, 256);
        return e;
    };
    rs_layer_weights o{};
    RS_HIP(copy(src->ln1_g, H * 2, &o.ln1_g));
    RS_HIP(copy(src->ln2_g, H * 2, &o.ln2_g));
    auto pack = [&](const void* m, int rows, int K, const void* gain, int mode, int p0, int p1, const void** slot) -> hipError_t {
        *slot = p;
        hipLaunchKernelGGL(pack_rows_kernel, dim3(rows / 32 * ((K + PACK_K - 1) / PACK_K)), dim3(256), 0, st, (const bf16*)m, (const bf16*)gain, reinterpret_cast<bf16*>(p), K,
                           mode, p0, p1, (int)aligned(m, 16));
        p += align_up((size_t)rows * K * 2, 256);
        return hipGetLastError();
    };
    // W_qkv with the first norm's gain folded into its columns
    RS_HIP(pack(src->w_qkv, c->qkv_dim, f.hidden, src->ln1_g, PACK_QKV_ROPE, f.head_dim, c->q_dim + c->kv_dim, &o.w_qkv));
    if (f.qkv_bias) {
        RS_HIP(copy(src->b_qkv, (size_t)c->qkv_dim * 2, &o.b_qkv));
    } else {
        p += align_up((size_t)c->qkv_dim * 2, 256);
    }
    RS_HIP(pack(src->w_o, f.hidden, c->q_dim, nullptr, PACK_IDENTITY, 0, 0, &o.w_o));
    // W_gate / W_up interleaved in 16-row blocks (one unit = 16 gate rows + their up rows), second norm gain folded in
    RS_HIP(pack(src->w_gate_up, 2 * f.mlp_inter, f.hidden, src->ln2_g, PACK_GATE_UP, f.mlp_inter, 0, &o.w_gate_up));
    RS_HIP(pack(src->w_down, f.hidden, f.mlp_inter, nullptr, PACK_IDENTITY, 0, 0, &o.w_down));
    *packed = o;
    return RS_OK;
}

size_t rs_kv_bytes(const rs_ctx* c, int n_layers, int capacity_tokens) {
    if (!c || n_layers <= 0 || capacity_tokens <= 0) return 0;
    const size_t cap = align_up((size_t)capacity_tokens, 64);
    const size_t plane = align_up(cap * c->kv_dim * 2, 256);
    return 2 * plane * n_layers;
}

rs_status rs_kv_alloc(rs_ctx* c, int n_layers, int capacity_tokens, void* dev_mem, size_t bytes, rs_kv** out) {
    if (!c || !out) return fail(RS_EINVAL, "ctx / out is null");
    *out = nullptr;
    if (n_layers <= 0 || capacity_tokens <= 0) return fail(RS_EINVAL, "n_layers and capacity_tokens must be positive");
    if (!dev_mem || !aligned(dev_mem, 256)) return fail(RS_EINVAL, "dev_mem must be a 256-byte aligned device pointer");
    const size_t need = rs_kv_bytes(c, n_layers, capacity_tokens);
    if (bytes < need) return fail(RS_EWORKSPACE, "KV slab has %zu bytes, need %zu", bytes, need);
    rs_kv* kv = new rs_kv();
    kv->ctx = c;
    kv->n_layers = n_layers;
    kv->cap = (int)align_up((size_t)capacity_tokens, 64);
    kv->base = reinterpret_cast<char*>(dev_mem);
    kv->k_bytes = align_up((size_t)kv->cap * c->kv_dim * 2, 256);
    kv->layer_bytes = 2 * kv->k_bytes;
    kv->len.assign(n_layers, 0);
    *out = kv;
    return RS_OK;
}

static bool fp8_scales_ok(float k_scale, float v_scale) {
    return k_scale > 0.0f && v_scale > 0.0f && std::isfinite(k_scale) && std::isfinite(v_scale) && std::isfinite(1.0f / k_scale) &&
           std::isfinite(1.0f / v_scale);
}

size_t rs_kv_fp8_bytes(const rs_ctx* c, int n_layers, int capacity_tokens) {
    if (!c || n_layers <= 0 || capacity_tokens <= 0) return 0;
    const size_t cap = align_up((size_t)capacity_tokens, 64);
    const size_t plane = align_up(cap * c->kv_dim, 256);
    return 2 * plane * n_layers;
}

rs_status rs_kv_alloc_fp8(rs_ctx* c, int n_layers, int capacity_tokens, float k_scale, float v_scale, void* dev_mem, size_t bytes,
                          rs_kv** out) {
    if (!c || !out) return fail(RS_EINVAL, "ctx / out is null");
    *out = nullptr;
    if (n_layers <= 0 || capacity_tokens <= 0) return fail(RS_EINVAL, "n_layers and capacity_tokens must be positive");
    if (!fp8_scales_ok(k_scale, v_scale))
        return fail(RS_EINVAL, "k_scale = %g and v_scale = %g must be positive, finite and have a finite reciprocal", k_scale, v_scale);
    if (!dev_mem || !aligned(dev_mem, 256)) return fail(RS_EINVAL, "dev_mem must be a 256-byte aligned device pointer");
    const size_t need = rs_kv_fp8_bytes(c, n_layers, capacity_tokens);
    if (bytes < need) return fail(RS_EWORKSPACE, "KV slab has %zu bytes, need %zu", bytes, need);
    rs_kv* kv = new rs_kv();
    kv->ctx = c;
    kv->n_layers = n_layers;
    kv->cap = (int)align_up((size_t)capacity_tokens, 64);
    kv->base = reinterpret_cast<char*>(dev_mem);
    kv->k_bytes = align_up((size_t)kv->cap * c->kv_dim, 256);
    kv->layer_bytes = 2 * kv->k_bytes;
    kv->len.assign(n_layers, 0);
    kv->fp8 = true;
    kv->k_scale = k_scale;
    kv->v_scale = v_scale;
    *out = kv;
    return RS_OK;
}

int rs_kv_is_fp8(const rs_kv* kv) { return kv ? (kv->fp8 ? 1 : 0) : -1; }

size_t rs_kv_page_bytes(const rs_ctx* c) {
    if (!c) return 0;
    return (size_t)2 * c->cfg.n_kv_heads * 64 * c->cfg.head_dim * 2;
}

size_t rs_kv_page_bytes_fp8(const rs_ctx* c) { return rs_kv_page_bytes(c) / 2; }

static rs_status pool_create(rs_ctx* c, void* dev_mem, size_t bytes, bool fp8, rs_kv_pool** out);
rs_status rs_kv_pool_create(rs_ctx* c, void* dev_mem, size_t bytes, rs_kv_pool** out) { return pool_create(c, dev_mem, bytes, false, out); }
rs_status rs_kv_pool_create_fp8(rs_ctx* c, void* dev_mem, size_t bytes, rs_kv_pool** out) { return pool_create(c, dev_mem, bytes, true, out); }
int rs_kv_pool_is_fp8(const rs_kv_pool* p) { return p ? (p->fp8 ? 1 : 0) : -1; }

static rs_status pool_create(rs_ctx* c, void* dev_mem, size_t bytes, bool fp8, rs_kv_pool** out) {
    if (!c || !out) return fail(RS_EINVAL, "ctx / out is null");
    *out = nullptr;
    if (!dev_mem || !aligned(dev_mem, 256)) return fail(RS_EINVAL, "dev_mem must be a 256-byte aligned device pointer");
    const size_t pb = fp8 ? rs_kv_page_bytes_fp8(c) : rs_kv_page_bytes(c);
    const size_t n = bytes / pb;
    if (n == 0) return fail(RS_EWORKSPACE, "the pool's memory (%zu bytes) is smaller than one page (%zu bytes)", bytes, pb);
    if (n > (size_t)0x7fffffff) return fail(RS_EINVAL, "more than 2^31 - 1 pages");
    rs_kv_pool* p = new rs_kv_pool();
    p->ctx = c;
    p->base = reinterpret_cast<char*>(dev_mem);
    p->page_bytes = pb;
    p->fp8 = fp8;
    p->n_pages = (int)n;
    p->free_pages.resize(n);
    for (size_t i = 0; i < n; ++i) p->free_pages[i] = (int)(n - 1 - i);  // page 0 is handed out first
    *out = p;
    return RS_OK;
}

rs_status rs_kv_pool_destroy(rs_kv_pool* p) {
    if (!p) return RS_OK;
    if (p->n_caches != 0) return fail(RS_ESTATE, "%d caches still use this pool", p->n_caches);
    delete p;
    return RS_OK;
}

int rs_kv_pool_pages(const rs_kv_pool* p) { return p ? p->n_pages : -1; }
int rs_kv_pool_free_pages(const rs_kv_pool* p) { return p ? (int)p->free_pages.size() : -1; }

static rs_status alloc_paged(rs_ctx* c, rs_kv_pool* pool, int n_layers, bool fp8, float k_scale, float v_scale, rs_kv** out);
rs_status rs_kv_alloc_paged(rs_ctx* c, rs_kv_pool* pool, int n_layers, rs_kv** out) {
    return alloc_paged(c, pool, n_layers, false, 1.0f, 1.0f, out);
}
rs_status rs_kv_alloc_paged_fp8(rs_ctx* c, rs_kv_pool* pool, int n_layers, float k_scale, float v_scale, rs_kv** out) {
    return alloc_paged(c, pool, n_layers, true, k_scale, v_scale, out);
}

static rs_status alloc_paged(rs_ctx* c, rs_kv_pool* pool, int n_layers, bool fp8, float k_scale, float v_scale, rs_kv** out) {
    if (!c || !out) return fail(RS_EINVAL, "ctx / out is null");
    *out = nullptr;
    if (!pool) return fail(RS_EINVAL, "pool is null");
    if (pool->ctx != c) return fail(RS_ESTATE, "the pool belongs to another context");
    if (pool->fp8 != fp8)
        return fail(RS_ESTATE, "the pool holds %s pages, the cache asked for is %s", pool->fp8 ? "8-bit" : "bfloat16", fp8 ? "8-bit" : "bfloat16");
    if (n_layers <= 0) return fail(RS_EINVAL, "n_layers must be positive");
    if (fp8 && !fp8_scales_ok(k_scale, v_scale))
        return fail(RS_EINVAL, "k_scale = %g and v_scale = %g must be positive, finite and have a finite reciprocal", k_scale, v_scale);
    rs_kv* kv = new rs_kv();
    kv->ctx = c;
    kv->n_layers = n_layers;
    kv->cap = 0;
    kv->base = nullptr;
    kv->k_bytes = kv->layer_bytes = 0;
    kv->len.assign(n_layers, 0);
    kv->pool = pool;
    kv->fp8 = fp8;
    kv->k_scale = k_scale;
    kv->v_scale = v_scale;
    kv->pages.assign(n_layers, std::vector<int>());
    ++pool->n_caches;
    *out = kv;
    return RS_OK;
}

void rs_kv_free(rs_kv* kv) {
    if (!kv) return;
    if (kv->paged()) {
        for (int l = 0; l < kv->n_layers; ++l) kv->give_back_pages(l, 0);
        --kv->pool->n_caches;
    }
    delete kv;
}

int rs_kv_len(const rs_kv* kv, int layer) {
    if (!kv || layer < 0 || layer >= kv->n_layers) return -1;
    return kv->len[layer];
}

int rs_kv_capacity(const rs_kv* kv) {
    if (!kv) return -1;
    if (!kv->paged()) return kv->cap;
    size_t fewest = kv->pages[0].size();
    for (const auto& pl : kv->pages) fewest = std::min(fewest, pl.size());
    return (int)(fewest * 64);
}

rs_status rs_kv_reset(rs_kv* kv) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    std::fill(kv->len.begin(), kv->len.end(), 0);
    if (kv->paged())
        for (int l = 0; l < kv->n_layers; ++l) kv->give_back_pages(l, 0);
    return RS_OK;
}

rs_status rs_kv_truncate(rs_kv* kv, int layer, int n_tokens) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    if (layer < 0 || layer >= kv->n_layers) return fail(RS_EINVAL, "layer %d out of range", layer);
    if (n_tokens < 0 || n_tokens > kv->len[layer]) return fail(RS_EINVAL, "n_tokens = %d outside [0, %d]", n_tokens, kv->len[layer]);
    kv->len[layer] = n_tokens;
    if (kv->paged()) kv->give_back_pages(layer, n_tokens);
    return RS_OK;
}

rs_status rs_kv_export(const rs_kv* kv, int layer, void* k_out, void* v_out, void* stream) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    if (layer < 0 || layer >= kv->n_layers) return fail(RS_EINVAL, "layer %d out of range", layer);
    const int n = kv->len[layer];
    if (n == 0) return RS_OK;
    if (!k_out || !v_out) return fail(RS_EINVAL, "k_out / v_out is null");
    if (!kv->ctx->has_device) return fail(RS_EHIP, "no HIP device");
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (kv->fp8) return fp8_export(kv, layer, (bf16*)k_out, (bf16*)v_out, st);
    for_each_kv_window(kv, layer, n, [&](const ReqDesc& rq, const KVPageWindow& win, int b0, int t0, int nt) {
        launch_export<bf16>(kv->ctx, rq, Fp8CacheDesc{}, win, b0, (bf16*)k_out, (bf16*)v_out, t0, nt, st);
    });
    RS_HIP(hipGetLastError());
    return RS_OK;
}

rs_status rs_kv_import(rs_kv* kv, int layer, const void* k, const void* v, int n_tokens, void* stream) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    {
        const rs_status s = import_check(kv, layer, n_tokens);
        if (s != RS_OK) return s;
    }
    if (n_tokens == 0) {
        kv->len[layer] = 0;
        if (kv->paged()) kv->give_back_pages(layer, 0);
        return RS_OK;
    }
    if (!k || !v) return fail(RS_EINVAL, "k / v is null");
    if (!kv->ctx->has_device) return fail(RS_EHIP, "no HIP device");
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (kv->paged()) {
        kv->take_pages(layer, n_tokens);
        kv->give_back_pages(layer, n_tokens);
    }
    if (kv->fp8) {
        const rs_status s = fp8_import(kv, layer, (const bf16*)k, (const bf16*)v, n_tokens, st);
        if (s == RS_OK) kv->len[layer] = n_tokens;
        return s;
    }
    for_each_kv_window(kv, layer, n_tokens, [&](const ReqDesc& rq, const KVPageWindow& win, int b0, int t0, int nt) {
        launch_import<bf16>(kv->ctx, rq, Fp8CacheDesc{}, win, b0, (const bf16*)k, (const bf16*)v, t0, nt, st);
    });
    RS_HIP(hipGetLastError());
    kv->len[layer] = n_tokens;
    return RS_OK;
}

rs_status rs_kv_export_codes(const rs_kv* kv, int layer, void* k_codes, void* v_codes, void* stream) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    if (!kv->fp8) return fail(RS_ESTATE, "not an 8-bit cache");
    if (layer < 0 || layer >= kv->n_layers) return fail(RS_EINVAL, "layer %d out of range", layer);
    if (kv->len[layer] == 0) return RS_OK;
    if (!k_codes || !v_codes) return fail(RS_EINVAL, "k_codes / v_codes is null");
    if (!kv->ctx->has_device) return fail(RS_EHIP, "no HIP device");
    return fp8_export(kv, layer, (uint8_t*)k_codes, (uint8_t*)v_codes, reinterpret_cast<hipStream_t>(stream));
}

rs_status rs_kv_import_codes(rs_kv* kv, int layer, const void* k_codes, const void* v_codes, int n_tokens, void* stream) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    if (!kv->fp8) return fail(RS_ESTATE, "not an 8-bit cache");
    {
        const rs_status s = import_check(kv, layer, n_tokens);
        if (s != RS_OK) return s;
    }
    if (n_tokens == 0) {
        kv->len[layer] = 0;
        if (kv->paged()) kv->give_back_pages(layer, 0);
        return RS_OK;
    }
    if (!k_codes || !v_codes) return fail(RS_EINVAL, "k_codes / v_codes is null");
    if (!kv->ctx->has_device) return fail(RS_EHIP, "no HIP device");
    if (kv->paged()) {
        kv->take_pages(layer, n_tokens);
        kv->give_back_pages(layer, n_tokens);
    }
    const rs_status s = fp8_import(kv, layer, (const uint8_t*)k_codes, (const uint8_t*)v_codes, n_tokens, reinterpret_cast<hipStream_t>(stream));
    if (s == RS_OK) kv->len[layer] = n_tokens;
    return s;
}

rs_status rs_profile_enable(rs_ctx* c, int step, int max_launches) {
    if (!c) return fail(RS_EINVAL, "ctx is null");
    if (step < -1 || step >= RS_STEP_COUNT) return fail(RS_EINVAL, "step %d out of range", step);
    if (step >= 0 && max_launches <= 0) return fail(RS_EINVAL, "max_launches must be positive");
    if (step >= 0 && !c->has_device) return fail(RS_EHIP, "no HIP device");
    c->prof_step = step;
    c->prof_count = 0;
    c->prof_seen = 0;
    c->prof_take = false;
    while (step >= 0 && (int)c->prof_events.size() < 2 * max_launches) {
        hipEvent_t e;
        RS_HIP(hipEventCreate(&e));
        c->prof_events.push_back(e);
    }
    return RS_OK;
}

rs_status rs_profile_sample_every(rs_ctx* c, int every) {
    if (!c) return fail(RS_EINVAL, "ctx is null");
    if (every <= 0) return fail(RS_EINVAL, "every = %d must be positive", every);
    c->prof_every = every;
    return RS_OK;
}

rs_status rs_profile_read(rs_ctx* c, double* total_ms, int* launches) {
    if (!c || !total_ms || !launches) return fail(RS_EINVAL, "null argument");
    double sum = 0.0;
    for (int i = 0; i < c->prof_count; ++i) {
        RS_HIP(hipEventSynchronize(c->prof_events[2 * i + 1]));
        float ms = 0.0f;
        RS_HIP(hipEventElapsedTime(&ms, c->prof_events[2 * i], c->prof_events[2 * i + 1]));
        sum += ms;
    }
    *total_ms = sum;
    *launches = c->prof_count;
    c->prof_count = 0;
    return RS_OK;
}

size_t rs_workspace_bytes(const rs_ctx* c, int max_tokens, int max_requests) {
    if (!c || max_tokens <= 0 || max_requests <= 0) return 0;
    return ws_layout(c, max_tokens, max_requests).total;
}

size_t rs_workspace_bytes_fp8kv(const rs_ctx* c, int max_tokens, int max_requests, size_t max_visible_tokens) {
    if (!c || max_tokens <= 0 || max_requests <= 0) return 0;
    // every request's share is rounded up to whole 64-token blocks
    return ws_layout(c, max_tokens, max_requests).total + fp8_expansion_bytes(c, (long)max_visible_tokens + 63L * max_requests);
}

rs_status rs_prefill_chunk(rs_ctx* ctx, const rs_layer_weights* packed, int layer, rs_kv* kv, const void* x, int T, void* y,
                           void* workspace, size_t workspace_bytes, void* stream) {
    if (!kv) return fail(RS_EINVAL, "kv is null");
    if (T < 0) return fail(RS_EINVAL, "T = %d is negative", T);
    rs_kv* kvs[1] = {kv};
    int lens[1] = {T};
    return prefill_impl(ctx, packed, layer, kvs, lens, 1, x, y, workspace, workspace_bytes, stream);
}

size_t rs_static_workspace_bytes(void) { return RS_STATIC_WORKSPACE_BYTES; }

rs_status rs_prefill_chunk_static(rs_ctx* ctx, const rs_layer_weights* packed, int layer, rs_kv* kv, const void* x, int T, void* y,
                                  void* stream) {
    if (!ctx) return fail(RS_EINVAL, "ctx is null");
    if (!kv) return fail(RS_EINVAL, "kv is null");
    if (T < 0) return fail(RS_EINVAL, "T = %d is negative", T);
    if (ctx->has_device) {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev != ctx->device)
            return fail(RS_ESTATE, "the current GPU (%d) is not the one the context was created on (%d)", dev, ctx->device);
    }
    // (a host-only context has no array to point at; every check before the missing device still runs, on a stand-in address)
    void* ws = ctx->has_device ? ctx->static_ws : reinterpret_cast<void*>(uintptr_t{256});
    rs_kv* kvs[1] = {kv};
    int lens[1] = {T};
    const rs_status s = prefill_impl(ctx, packed, layer, kvs, lens, 1, x, y, ws, RS_STATIC_WORKSPACE_BYTES, stream);
    if (s == RS_EWORKSPACE) {
        const std::string why = g_last_error;
        return fail(RS_EWORKSPACE, "%s: beyond the static workspace of rs_prefill_chunk_static (use rs_prefill_chunk with a workspace of the caller's)",
                    why.c_str());
    }
    return s;
}

rs_status rs_prefill_batch(rs_ctx* ctx, const rs_layer_weights* packed, int layer, rs_kv* const* kvs, const int* chunk_lens, int R,
                           const void* x, void* y, void* workspace, size_t workspace_bytes, void* stream) {
    return prefill_impl(ctx, packed, layer, kvs, chunk_lens, R, x, y, workspace, workspace_bytes, stream);
}

rs_status rs_ctx_set_mrope_sections(rs_ctx* c, int temporal, int height, int width) {
    if (!c) return fail(RS_EINVAL, "ctx is null");
    if (temporal < 0 || height < 0 || width < 0 || temporal + height + width != c->cfg.head_dim / 2)
        return fail(RS_EINVAL, "sections %d + %d + %d must be non-negative and sum to head_dim / 2 = %d", temporal, height, width,
                    c->cfg.head_dim / 2);
    if (temporal % 4 || height % 4 || width % 4) return fail(RS_EINVAL, "each section must be a multiple of 4 rotary pairs");
    c->mrope_b0 = temporal;
    c->mrope_b1 = temporal + height;
    return RS_OK;
}

rs_status rs_prefill_batch_mrope(rs_ctx* ctx, const rs_layer_weights* packed, int layer, rs_kv* const* kvs, const int* chunk_lens,
                                 int R, const int* positions, const void* x, void* y, void* workspace, size_t workspace_bytes,
                                 void* stream) {
    if (!positions) return fail(RS_EINVAL, "positions is null");
    return prefill_impl(ctx, packed, layer, kvs, chunk_lens, R, x, y, workspace, workspace_bytes, stream, positions);
}

static rs_status model_batch(rs_ctx* ctx, const rs_layer_weights* packed_layers, int n_layers, rs_kv* const* kvs, const int* chunk_lens,
                             int R, const int* positions3, const void* x, void* y, void* workspace, size_t workspace_bytes,
                             void* stream) {
    if (!packed_layers) return fail(RS_EINVAL, "packed_layers is null");
    if (n_layers <= 0) return fail(RS_EINVAL, "n_layers = %d must be positive", n_layers);
    int T = 0;
    PoolNeed need;
    for (int l = 0; l < n_layers; ++l) {  // all checks first: a failing call leaves every cache untouched
        const rs_status s = prefill_check(ctx, &packed_layers[l], l, kvs, chunk_lens, R, x, y, workspace, workspace_bytes, &T,
                                          positions3, &need);
        if (s != RS_OK) return s;
    }
    {
        const rs_status s = check_need(need);  // paged caches: the pages of all layers together must be there
        if (s != RS_OK) return s;
    }
    if (T > 0 && !ctx->has_device) return fail(RS_EHIP, "no HIP device: the context was created on a host without a GPU");
    if (T == 0) return RS_OK;
    // Layer 0 reads x; later layers work on y in place.  Between two layers the split-K sum of the down projection, the
    // pass that takes the next layer's norm factors and the copy into its GEMMs' operand layout are one kernel (see
    // rms_and_fragment_major_kernel with planes): the bits are those of the layers called one by one.
    // The attention plan of one layer serves the next while their caches are equally long (planning takes 2 to 15 us of host
    // time, of about 30 per layer).
    PendingReduce pending;
    AttnPlanCache plans;
    for (int l = 0; l < n_layers; ++l) {
        PendingReduce next;
        const rs_status s = prefill_enqueue(ctx, &packed_layers[l], l, kvs, chunk_lens, R, T, l == 0 ? x : y, y, workspace, stream,
                                            plans, positions3, l > 0 ? &pending : nullptr, l + 1 < n_layers ? &next : nullptr);
        if (s != RS_OK) return s;
        pending = next;
    }
    return RS_OK;
}

rs_status rs_prefill_model_batch(rs_ctx* ctx, const rs_layer_weights* packed_layers, int n_layers, rs_kv* const* kvs,
                                 const int* chunk_lens, int R, const void* x, void* y, void* workspace, size_t workspace_bytes,
                                 void* stream) {
    return model_batch(ctx, packed_layers, n_layers, kvs, chunk_lens, R, nullptr, x, y, workspace, workspace_bytes, stream);
}

rs_status rs_prefill_model_batch_mrope(rs_ctx* ctx, const rs_layer_weights* packed_layers, int n_layers, rs_kv* const* kvs,
                                       const int* chunk_lens, int R, const int* positions, const void* x, void* y, void* workspace,
                                       size_t workspace_bytes, void* stream) {
    if (!positions) return fail(RS_EINVAL, "positions is null");
    return model_batch(ctx, packed_layers, n_layers, kvs, chunk_lens, R, positions, x, y, workspace, workspace_bytes, stream);
}

static size_t lm_head_bytes_f32(const rs_ctx* c, int n_rows) { return align_up((size_t)n_rows * c->cfg.hidden * 4, 256); }
static size_t lm_head_bytes_split(const rs_ctx* c, int n_rows) {
    return (size_t)((n_rows + LM_GROUP - 1) / LM_GROUP) * c->cfg.hidden * 64;   // 32 bfloat16 columns per group of rows
}

size_t rs_lm_head_workspace_bytes(const rs_ctx* c, int n_rows) {
    if (!c || n_rows <= 0) return 0;
    return std::max(lm_head_bytes_f32(c, n_rows), n_rows >= LM_MFMA_ROWS ? lm_head_bytes_split(c, n_rows) : 0);
}

rs_status rs_lm_head(rs_ctx* c, const void* final_norm_gain, const void* w_lm, int vocab, const void* x, int n_rows, void* logits,
                     void* workspace, size_t workspace_bytes, void* stream) {
    if (!c) return fail(RS_EINVAL, "ctx is null");
    if (n_rows < 0) return fail(RS_EINVAL, "n_rows = %d is negative", n_rows);
    if (vocab <= 0) return fail(RS_EINVAL, "vocab = %d must be positive", vocab);
    if (n_rows == 0) return RS_OK;
    if (!final_norm_gain || !w_lm || !x || !logits || !workspace) return fail(RS_EINVAL, "null argument");
    if (!aligned(final_norm_gain, 16) || !aligned(w_lm, 16) || !aligned(x, 16) || !aligned(logits, 4) || !aligned(workspace, 256))
        return fail(RS_EINVAL, "misaligned argument");
    if (workspace_bytes < lm_head_bytes_f32(c, n_rows))
        return fail(RS_EWORKSPACE, "workspace has %zu bytes, this call needs %zu", workspace_bytes, lm_head_bytes_f32(c, n_rows));
    // the kernel keeps its group of normalised rows (fp32) in LDS: as many rows per launch, up to LM_ROWS, as 160 KB hold
    constexpr size_t LDS_BYTES = 160 * 1024;
    const int H = c->cfg.hidden;
    if ((size_t)H * 4 > LDS_BYTES) return fail(RS_EINVAL, "hidden = %d: one fp32 row does not fit the %zu bytes of LDS the head kernel stages it in", H, LDS_BYTES);
    if (!c->has_device) return fail(RS_EHIP, "no HIP device");
    if (c->lm_rows == 0) {  // first use on this context: opt in to the LDS size once
        const int rows = (int)std::min<size_t>(LM_ROWS, LDS_BYTES / ((size_t)H * 4));
        RS_HIP(hipFuncSetAttribute((const void*)lm_head_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, rows * H * 4));
        RS_HIP(hipFuncSetAttribute((const void*)lm_head_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, rows * H * 4));
        c->lm_rows = rows;
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    // Three rows and more go through the matrix pipe, up to 20 per pass over the vocabulary.  One or two, which the LDS kernel
    // streams as fast (170 and 177 us on 152064 x 3584, against 182), and a workspace of 4 H bytes per row, which holds no
    // split rows, take that kernel.
    const size_t w_bytes = (size_t)vocab * H * 2;
    const bool once = w_bytes >= LM_STREAM_BYTES;
    if (n_rows >= LM_MFMA_ROWS && workspace_bytes >= lm_head_bytes_split(c, n_rows)) {
        bf16* hb = reinterpret_cast<bf16*>(workspace);
        hipLaunchKernelGGL(final_norm_split_kernel, dim3(LM_GROUP + 1, (n_rows + LM_GROUP - 1) / LM_GROUP), dim3(256), 0, st, (const bf16*)x,
                           (const bf16*)final_norm_gain, hb, n_rows, H, c->cfg.rms_eps);
        RS_HIP(hipGetLastError());
        // (one workgroup per compute unit; more if a share would not fit the kernel's 32-bit offsets)
        const dim3 grid((unsigned)std::min<size_t>(std::max<size_t>(c->n_cu, (w_bytes >> 30) + 1), (vocab + LM_VROWS - 1) / LM_VROWS));
        for (int r0 = 0; r0 < n_rows; r0 += LM_MAX_GROUPS * LM_GROUP) {
            const int R = std::min(LM_MAX_GROUPS * LM_GROUP, n_rows - r0), groups = (R + LM_GROUP - 1) / LM_GROUP;
            const bf16* hg = hb + (size_t)(r0 / LM_GROUP) * H * 32;
            float* lg = reinterpret_cast<float*>(logits) + (size_t)r0 * vocab;
            const auto launch = [&](auto ng) {
                if (once) hipLaunchKernelGGL((lm_head_mfma_kernel<decltype(ng)::value, true>), grid, dim3(256), 0, st, (const bf16*)w_lm, hg, lg, R, vocab, H);
                else hipLaunchKernelGGL((lm_head_mfma_kernel<decltype(ng)::value, false>), grid, dim3(256), 0, st, (const bf16*)w_lm, hg, lg, R, vocab, H);
            };
            if (groups == 1) launch(std::integral_constant<int, 1>{});
            else launch(std::integral_constant<int, 2>{});
            RS_HIP(hipGetLastError());
        }
        return RS_OK;
    }
    float* h = reinterpret_cast<float*>(workspace);
    hipLaunchKernelGGL(final_norm_kernel, dim3((n_rows + 3) / 4), dim3(256), 0, st, (const bf16*)x, (const bf16*)final_norm_gain, h,
                       n_rows, H, c->cfg.rms_eps);
    RS_HIP(hipGetLastError());
    const int blocks = std::min(4 * c->n_cu, (vocab + 4 * LM_VGROUP - 1) / (4 * LM_VGROUP));
    for (int r0 = 0; r0 < n_rows; r0 += c->lm_rows) {  // the vocabulary matrix is streamed once per group of rows
        const int R = std::min(c->lm_rows, n_rows - r0);
        hipLaunchKernelGGL(once ? lm_head_kernel<true> : lm_head_kernel<false>, dim3(blocks), dim3(256), (size_t)R * H * 4, st, (const bf16*)w_lm, (const float*)(h + (size_t)r0 * H),
                           reinterpret_cast<float*>(logits) + (size_t)r0 * vocab, R, vocab, H);
        RS_HIP(hipGetLastError());
    }
    return RS_OK;
}

}  // extern "C"
