// Host side of libstpi: argument validation, filter taps, kernel selection,
// workspace layout and the C ABI declared in include/stpi.h.
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

#include "../../include/stpi.h"
#include "dtype_ops.hpp"
#include "host_internal.hpp"

namespace stpi {

static thread_local std::string g_last_error;

int fail(int status, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return status;
}

int hip_fail(hipError_t e, const char *where) {
    return fail(STPI_EHIP, "%s: %s", where, hipGetErrorString(e));
}

void clear_error() { g_last_error.clear(); }

const DtypeOps *ops_for(int dtype) {
    switch (dtype) {
        case STPI_F32: return dtype_ops_f32();
        case STPI_BF16: return dtype_ops_bf16();
        case STPI_F64: return dtype_ops_f64();
        default: return nullptr;
    }
}

int validate_problem(const stpi_problem *p) {
    if (!p) return fail(STPI_EINVAL, "problem is NULL");
    if (p->T < 1 || p->H < 1 || p->W < 1)
        return fail(STPI_EINVAL, "volume must be at least 1x1x1 (got %dx%dx%d)", p->T, p->H, p->W);
    if (!(p->sigma_s > 0.0f) || !(p->sigma_t > 0.0f) || !std::isfinite(p->sigma_s) || !std::isfinite(p->sigma_t))
        return fail(STPI_EINVAL, "sigmas must be finite and > 0");
    if (p->r_s < 0 || p->r_t < 0) return fail(STPI_EINVAL, "radii must be >= 0");
    if (p->r_s > STPI_MAX_RS || p->r_t > STPI_MAX_RT)
        return fail(STPI_EUNSUPPORTED, "radii (%d, %d) exceed the compiled maximum (%d, %d)", p->r_s, p->r_t,
                    STPI_MAX_RS, STPI_MAX_RT);
    if (!ops_for(p->dtype)) return fail(STPI_EINVAL, "unknown dtype %d", p->dtype);
    if ((int64_t)p->H * p->W > (int64_t)1 << 30)
        return fail(STPI_EUNSUPPORTED, "frame of %d x %d voxels is too large", p->H, p->W);
    return STPI_OK;
}

// Taps exp(-d^2 / (2 sigma^2)) for |d| <= r, centred at index 16 (space) / 8
// (time), zero beyond the radius. The centre tap is 1 (unnormalised kernel).
void make_taps(const stpi_problem *p, double *gs, double *gt) {
    for (int i = 0; i < 2 * 16 + 1; ++i) gs[i] = 0.0;
    for (int i = 0; i < 2 * 8 + 1; ++i) gt[i] = 0.0;
    const double ss = (double)p->sigma_s, stt = (double)p->sigma_t;
    for (int d = -p->r_s; d <= p->r_s; ++d) gs[d + 16] = std::exp(-(double)(d * d) / (2.0 * ss * ss));
    for (int d = -p->r_t; d <= p->r_t; ++d) gt[d + 8] = std::exp(-(double)(d * d) / (2.0 * stt * stt));
}

static double variant_cost(const Variant &v, const stpi_problem *p) {
    // Taps per voxel plus the y-pass over the x-halo, on the padded tile grid.
    const double gx = std::ceil((double)p->W / v.TW), gy = std::ceil((double)p->H / v.TH);
    const double cover = gx * v.TW * gy * v.TH / ((double)p->W * p->H);
    if (v.PIPE == 3) {
        // matrix-core spatial passes (chains in product form): bound by memory
        // traffic and latency, not by the space radius; in the units of the
        // tap count below, measured at 480 x 854 frames as 42 (margin 16) or
        // 30 (margin 8) plus two per temporal tap, 10% less where two
        // workgroups share a CU
        const double base = v.RS > 8 ? 42.0 : 30.0;
        const double occ = v.blocks_per_cu() >= 2 ? 0.9 : 1.0;
        return (base + 2.0 * (2.0 * v.RT + 1)) * cover * occ;
    }
    const double taps = (2.0 * v.RS + 1) * (1.0 + 2.0 * v.RS / v.TW) + (2.0 * v.RS + 1) + (2.0 * v.RT + 1);
    return taps * cover;
}

static int tiles_for(const Variant &v, const stpi_problem *p) {
    return ((p->W + v.TW - 1) / v.TW) * ((p->H + v.TH - 1) / v.TH);
}

// Whether a loop with a workgroup per tile and output frame (PIPE 4) beats the
// streamed loops. It costs about 5.5 us plus 7 us per thousand 16 x 64 tiles
// and frames (it re-reads 2 r_t + 1 frames for each), a streamed step 8 us plus
// about a third of a microsecond per frame of its segments. Measured at r =
// (4, 2), chain step in us, streamed / 8 x 32 / 16 x 64 tile: 8x64x112 10.3 / 5.8 /
// 6.7 (256 and 64 workgroups), 64x48x64 15.4 / 7.5 / 6.4 (768, 192), 16x120x214
// 12.3 / 12.6 / 9.0 (1680, 512), 32x120x214 13.1 / 18.7 / 12.1 (3360, 1024),
// 2x480x854 9.1 / 18.0 / 11.2 (3240, 840); streamed / 16 x 64: 8x240x432 11.3 /
// 12.3 (840), 12x200x300 12.2 / 11.9 (780), 24x120x216 12.4 / 10.5 (768),
// 128x64x112 23.2 / 11.1 (1024), 10x230x432 12.0 / 14.8 (1050). So: the small
// tile while every workgroup has a CU of its own, the large one up to two per CU
// on clips longer than the temporal window and up to four per CU on clips of
// more than twice that. The other types lie alike (streamed / 8 x 32 / 16 x 64),
// bfloat16: 8x64x112 10.7 / 5.6 / 6.6, 16x120x214 10.9 / 12.1 / 8.4, 128x64x112 24.0 /
// 19.9 / 10.2, 8x240x432 10.9 / 18.4 / 11.1, 10x230x432 11.9 / 20.7 / 13.3; double:
// 13.2 / 6.1 / 8.1, 14.8 / 16.6 / 12.4, 31.4 / 27.1 / 16.2, 15.2 / 25.5 / 18.2, 16.3 /
// 28.6 / 22.1, and 12x200x300 16.6 / 22.2 / 16.6.
bool gather_pays(const Variant &v, const stpi_problem *p) {
    const int64_t units = (int64_t)tiles_for(v, p) * p->T;
    if (v.TH * v.TW <= 256) return units <= device_cus();
    return (units <= 2 * device_cus() && p->T > 2 * v.RT) || (units <= 4 * device_cus() && p->T > 4 * v.RT);
}

// Relative duration of a step on one of the matrix-core tiles of a margin: the
// phases of its slowest frame segment times the cost of a phase. A wide tile
// (32 x 128 or 64 x 64, one workgroup per CU) counts 1 per phase. A 32 x 64 tile
// (two per CU) has half the work in a phase and more halo: it wins while its
// workgroups have a CU each, and is about even with the wide tile where two
// share one, better while the chain's three volumes stay in the 256 MB
// last-level cache and worse when the larger halo comes from HBM. Measured, us
// per chain step, wide / 32 x 64: float, r = (8, 3): 21x233x347 27.8 / 19.8,
// 32x240x432 27.8 / 26.7, 64x360x640 46.6 / 43.9, 64x480x854 90.6 / 96.4,
// 96x480x854 130 / 146; bfloat16, r = (15, 5): 21x233x347 41.8 / 34.6,
// 32x240x432 48.3 / 40.6, 16x480x854 36.3 / 42.1, 64x480x854 82.2 / 85.5.
static double mfma_tile_cost(const Variant &v, const stpi_problem *p) {
    const int nseg = segments_for(v, p);
    const long units = (long)tiles_for(v, p) * nseg, cus = device_cus();
    const int per_cu = v.blocks_per_cu();
    const double rounds = std::ceil((double)units / (double)(cus * per_cu));
    double phase = v.TH >= 64 ? 1.02 : 1.0;  // 64 x 64 behind 32 x 128 by 1 to 3% at every size measured
    if (per_cu >= 2) {
        const double bytes = 3.0 * p->T * p->H * p->W * (double)ops_for(p->dtype)->elem;
        if (v.RS > 8) phase = units <= cus ? 0.84 : 1.04;
        else phase = units <= cus ? 0.71 : bytes > 256.0 * 1024 * 1024 ? 1.06 : 0.95;
    }
    return segment_phases(p->T, v.RT, nseg) * rounds * phase;
}

// tape: a step of a differentiated pass. It runs on the vector units and keeps
// one order of its float sums at every size (streamed frames, base_segments):
// small gradients that are differences of large sums, such as the bias's, move by
// their own rounding with that order, more than float gradients of the same
// problem should between two sizes' paths.
const Variant *choose_variant(const stpi_problem *p, int forced_index, bool tape) {
    const bool allow_mfma = !tape;
    const DtypeOps *ops = ops_for(p->dtype);
    if (forced_index >= 0 && forced_index < ops->nvariants && !allow_mfma && ops->variants[forced_index].PIPE == 3)
        forced_index = -1;
    if (forced_index >= 0) {
        if (forced_index >= ops->nvariants) return nullptr;
        const Variant &v = ops->variants[forced_index];
        if (v.RS < p->r_s || v.RT < p->r_t) return nullptr;
        return &v;
    }
    int tuned = tuned_variant(p);
    if (tuned >= 0 && tuned < ops->nvariants) {
        const Variant &v = ops->variants[tuned];
        if (v.RS >= p->r_s && v.RT >= p->r_t && (!tape || v.PIPE < 3)) return &v;
    }
    const Variant *best = nullptr;
    double best_cost = 1e300;
    for (int i = 0; i < ops->nvariants; ++i) {
        const Variant &v = ops->variants[i];
        if (v.RS < p->r_s || v.RT < p->r_t) continue;
        if (v.PIPE == 3 && !allow_mfma) continue;
        if (v.PIPE == 4) {
            if (!tape && gather_pays(v, p)) return &v;
            continue;
        }
        const double c = variant_cost(v, p);
        if (c < best_cost) {
            best_cost = c;
            best = &v;
        }
    }
    if (!best || best->PIPE != 3) return best;
    // the tile among the matrix-core variants of the same radii
    const Variant *tile = best;
    double tile_cost = mfma_tile_cost(*best, p);
    for (int i = 0; i < ops->nvariants; ++i) {
        const Variant &v = ops->variants[i];
        if (v.PIPE != 3 || v.RS != best->RS || v.RT != best->RT) continue;
        const double c = mfma_tile_cost(v, p);
        if (c < tile_cost) {
            tile_cost = c;
            tile = &v;
        }
    }
    return tile;
}

int device_cus() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        hipDeviceProp_t prop;
        cus[dev] = hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0
                       ? prop.multiProcessorCount
                       : 256;
    }
    return cus[dev];
}

// Phases of the slowest of k frame segments of a T-frame tile: the frame walk
// of the tile loops (FrameWalk: RT input frames staged beyond each inner
// boundary, the last segment walked backward when it starts after frame 0)
// plus the 2 phases that fill the pipeline.
int segment_phases(int T, int RT, int k) {
    int worst = 0;
    for (int s = 0; s < k; ++s) {
        const int t0 = (int)((long)s * T / k), t1 = (int)((long)(s + 1) * T / k);
        const int ts = std::max(t0 - RT, 0), te = std::min(t1 + RT, T);
        const bool rev = t1 == T && t0 > 0;
        worst = std::max(worst, (rev ? te - t0 : t1 - ts) + RT + 2);
    }
    return worst;
}

// Segments per tile beyond the `from` that the rules below give: while every
// segment can have a CU of its own, the step takes as long as its slowest
// segment, so the frames are split further where that lowers the phase count (a
// whole tile also ends with RT epilogue-only phases that a split with a backward
// last segment avoids; short clips, e.g. the windows of an online run, gain
// most). What the added segments re-stage runs on CUs that were idle. Measured,
// us per chain step before / after: float r = (15, 5) 24x90x108 45.3 / 34.7 (1
// segment / 4), 32x240x432 52.0 / 38.5 (3 / 8), 96x270x480 81.3 / 60.4 (4 / 7),
// 64x360x640 75.2 / 65.0 (3 / 4); r = (8, 3) 21x233x347 19.8 / 18.5 (3 / 4),
// 96x270x480 54.0 / 42.5 (4 / 7); bfloat16 r = (15, 5) 32x240x432 40.5 / 36.0.
int split_short_tiles(int tiles, int T, int RT, int from) {
    const int cus = device_cus();
    const int kmax = std::min(std::min(cus / tiles, STPI_NSEG_MAX), T);
    // more segments only for at least two phases fewer (each adds a
    // workgroup that re-stages RT frames)
    int best = from;
    for (int k = from + 1; k <= kmax; ++k)
        if (segment_phases(T, RT, k) + 1 < segment_phases(T, RT, best)) best = k;
    return best;
}

// Frame segments per tile. When a clip has fewer tiles than the chip holds
// resident workgroups, each tile's frames are split so that more workgroups
// (with independent barriers) share every CU. A segment re-reads and
// re-filters RT input frames on each inner side, so segments are normally at
// least 4 RT frames long and at most 4 per tile. A launch that would still
// fill less than half of the resident slots (a small clip, e.g. a coarse
// level of a two-level start) is bound by the frame-after-frame latency of
// its few workgroups, not by work: there segments may be as short as 2 RT
// frames and up to STPI_NSEG_MAX per tile.
static int base_segments(const Variant &v, const stpi_problem *p) {
    const int tiles = tiles_for(v, p);
    const int resident = device_cus() * v.blocks_per_cu();
    const int rt = v.RT > 0 ? v.RT : 1;
    const int fit = resident / tiles;
    int nseg = std::min(std::min(fit, p->T / (4 * rt)), 4);
    if (nseg < 1) nseg = 1;
    if ((long)tiles * nseg * 2 <= resident) {
        const int small = std::min(std::min(fit, p->T / (2 * rt)), STPI_NSEG_MAX);
        if (small > nseg) nseg = small;
    }
    return nseg;
}

// Segments of a PIPE 4 launch: single frames, or as many as give the chip four
// workgroups per CU (such launches are only asked for by index).
static int gather_segments(const Variant &v, const stpi_problem *p) {
    return std::min(p->T, std::max(1, 4 * device_cus() / tiles_for(v, p)));
}

int segments_for(const Variant &v, const stpi_problem *p) {
    if (v.PIPE == 4) return gather_segments(v, p);
    return split_short_tiles(tiles_for(v, p), p->T, v.RT, base_segments(v, p));
}

int tape_segments(const Variant &v, const stpi_problem *p) {
    if (v.PIPE == 4) return gather_segments(v, p);
    const int nseg = base_segments(v, p);
    return nseg == 1 ? split_short_tiles(tiles_for(v, p), p->T, v.RT) : nseg;
}

int grid_blocks(const Variant &v, const stpi_problem *p) { return tiles_for(v, p) * segments_for(v, p); }
int tape_blocks(const Variant &v, const stpi_problem *p) { return tiles_for(v, p) * tape_segments(v, p); }

// Workspace: [3 state slots][2 x partial sums][2 x maxima][ping-pong volume].
// A partials set holds the largest grid any compiled variant can use for this
// frame size, whatever the radii.
size_t partials_capacity(const stpi_problem *p) {
    const DtypeOps *ops = ops_for(p->dtype);
    size_t cap = (size_t)NORM_BLOCKS_HOST;
    for (int i = 0; i < ops->nvariants; ++i) {
        const Variant &v = ops->variants[i];
        const size_t g = (size_t)tiles_for(v, p) * (size_t)(v.PIPE == 4 ? gather_segments(v, p) : STPI_NSEG_MAX);
        if (g > cap) cap = g;
    }
    for (int i = 0; i < ops->nadj; ++i) {
        const AdjVariant &v = ops->adj_variants[i];
        const size_t g = (size_t)(((p->W + v.TW - 1) / v.TW) * ((p->H + v.TH - 1) / v.TH)) * STPI_NSEG_MAX;
        if (g > cap) cap = g;
    }
    return cap;
}

WsLayout layout_for(const stpi_problem *p) {
    WsLayout L;
    const DtypeOps *ops = ops_for(p->dtype);
    const size_t N = (size_t)p->T * p->H * p->W;
    L.state_off = 0;
    L.partials_off = (FINAL_SLOT + 1) * STATE_SLOT;
    L.partials_cap = partials_capacity(p);
    L.wmax_off = L.partials_off + 2 * L.partials_cap * 2 * sizeof(double);
    size_t off = L.wmax_off + 2 * L.partials_cap * sizeof(uint32_t);
    off = (off + 255) & ~(size_t)255;
    L.buf_off = off;
    L.total = off + ((N * ops->elem + 255) & ~(size_t)255);
    return L;
}

ChainMem chain_mem(const WsLayout &L, void *ws) {
    char *w = (char *)ws;
    return {(DevState *)(w + L.state_off), (double *)(w + L.partials_off), (uint32_t *)(w + L.wmax_off),
            L.partials_cap, w + L.buf_off};
}

static int g_forced_variant = -1;

// Captured iteration chains, keyed by every argument that shapes the launch
// sequence. Replaying a graph removes the per-launch host overhead of the chain's
// kernels (one per step, two where the steps are finalised by a launch of their
// own, and up to five around them).
struct GraphKey {
    stpi_problem p;
    const void *f;
    void *x, *ws;
    int init, max_iters;
    double tol;
    const Variant *v;
    hipStream_t s;
    int part;   // ChainPart
    int pform;  // product-form chain
    int defer;  // steps finalised by the next launch: the parts of a chain have to agree on it
    bool operator==(const GraphKey &o) const {
        return std::memcmp(&p, &o.p, sizeof(p)) == 0 && f == o.f && x == o.x && ws == o.ws && init == o.init &&
               max_iters == o.max_iters && tol == o.tol && v == o.v && s == o.s && part == o.part &&
               pform == o.pform && defer == o.defer;
    }
};
struct GraphEntry {
    GraphKey key;
    hipGraphExec_t exec;
    hipEvent_t launched;  // recorded after every launch: eviction waits for it
    unsigned long long last_use;
};
static std::mutex g_graph_mu;
static std::vector<GraphEntry> g_graphs;
static unsigned long long g_graph_clock = 0;
constexpr size_t GRAPH_CACHE_MAX = 16;

// STPI_NO_FUSE=1 finalises every step in a kernel of its own (for comparison).
bool fusion_disabled() {
    const char *e = std::getenv("STPI_NO_FUSE");
    return e && e[0] == '1';
}

static bool graphs_enabled() {
    const char *e = std::getenv("STPI_NO_GRAPH");
    return !(e && e[0] == '1');
}

// Chains on a matrix-core variant run in product form (one staged array per
// step) unless STPI_NO_PRODUCT=1; a chain of no steps keeps the plain form.
int chain_pform(const Variant *v, int max_iters) {
    const char *e = std::getenv("STPI_NO_PRODUCT");
    return v && v->launch_p && max_iters > 0 && !(e && e[0] == '1') ? 1 : 0;
}

int forced_variant() { return g_forced_variant; }
void set_forced_variant(int v) { g_forced_variant = v; }

enum ChainPart { CHAIN_ALL = 0, CHAIN_HEAD = 1, CHAIN_CHUNK_PART = 2, CHAIN_TAIL = 3 };

struct ChainArgs {
    const stpi_problem *p;
    const DtypeOps *ops;
    const Variant *v;
    const void *f;
    void *x;
    ChainMem m;
    int init, max_iters;
    double tol;
    int pform, defer;
};

int enqueue_chain_part(const ChainArgs &a, int part, hipStream_t s) {
    switch (part) {
        case CHAIN_ALL:
            return enqueue_iteration(a.p, a.ops, a.v, a.f, a.x, a.m, a.init, a.max_iters, a.tol, s, a.pform, a.defer);
        case CHAIN_HEAD: {
            const int rc = enqueue_chain_init(a.p, a.ops, a.x, a.m, a.init, a.max_iters, a.tol, s, a.v, a.f, a.pform);
            return rc ? rc : enqueue_chain_steps(a.p, a.v, a.f, a.x, a.m, CHAIN_CHUNK, s, a.pform, a.defer);
        }
        case CHAIN_CHUNK_PART:
            return enqueue_chain_steps(a.p, a.v, a.f, a.x, a.m, CHAIN_CHUNK, s, a.pform, a.defer);
        default:  // after whole segments
            return enqueue_chain_tail(a.p, a.ops, a.v, a.f, a.x, a.m, CHAIN_CHUNK, s, a.pform, a.defer);
    }
}

// Launches the cached graph for key, capturing `enqueue` into a new one on a miss.
// A graph may still be queued when its entry is evicted (callers need not
// synchronise between calls), so every launch records the entry's event and
// eviction waits for it before destroying the executable graph.
template <class F>
int launch_cached_graph(const GraphKey &key, F &&enqueue, hipStream_t s) {
    hipGraphExec_t exec = nullptr;
    hipEvent_t launched = nullptr;
    hipError_t e;
    {
        std::lock_guard<std::mutex> lk(g_graph_mu);
        for (auto &g : g_graphs)
            if (g.key == key) {
                exec = g.exec;
                launched = g.launched;
                g.last_use = ++g_graph_clock;
                // launch under the lock: no other thread can evict the entry in between
                if ((e = hipGraphLaunch(exec, s)) != hipSuccess) return hip_fail(e, "graph launch");
                if ((e = hipEventRecord(launched, s)) != hipSuccess) return hip_fail(e, "graph event");
                return STPI_OK;
            }
    }
    if (!exec) {
        if ((e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal)) != hipSuccess)
            return hip_fail(e, "begin capture");
        const int rc = enqueue();
        hipGraph_t graph = nullptr;
        e = hipStreamEndCapture(s, &graph);
        if (rc) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc;
        }
        if (e != hipSuccess) return hip_fail(e, "end capture");
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return hip_fail(e, "graph instantiate");
        if ((e = hipEventCreateWithFlags(&launched, hipEventDisableTiming)) != hipSuccess) {
            (void)hipGraphExecDestroy(exec);
            return hip_fail(e, "graph event");
        }
        std::lock_guard<std::mutex> lk(g_graph_mu);
        if (g_graphs.size() >= GRAPH_CACHE_MAX) {
            size_t old = 0;
            for (size_t i = 1; i < g_graphs.size(); ++i)
                if (g_graphs[i].last_use < g_graphs[old].last_use) old = i;
            (void)hipEventSynchronize(g_graphs[old].launched);
            (void)hipGraphExecDestroy(g_graphs[old].exec);
            (void)hipEventDestroy(g_graphs[old].launched);
            g_graphs.erase(g_graphs.begin() + old);
        }
        g_graphs.push_back(GraphEntry{key, exec, launched, ++g_graph_clock});
        if ((e = hipGraphLaunch(exec, s)) != hipSuccess) return hip_fail(e, "graph launch");
        if ((e = hipEventRecord(launched, s)) != hipSuccess) return hip_fail(e, "graph event");
    }
    return STPI_OK;
}

// Host-visible copy of the iteration state for the stop-flag poll (pinned,
// one per thread, kept for the life of the process), and its event.
DevState *pinned_state() {
    thread_local DevState *buf = nullptr;
    if (!buf && hipHostMalloc((void **)&buf, sizeof(DevState), hipHostMallocDefault) != hipSuccess) buf = nullptr;
    return buf;
}

hipEvent_t poll_event() {
    thread_local hipEvent_t ev = nullptr;
    if (!ev && hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) ev = nullptr;
    return ev;
}

}  // namespace stpi

using namespace stpi;

extern "C" {

const char *stpi_status_string(int status) {
    switch (status) {
        case STPI_OK: return "ok";
        case STPI_EINVAL: return "invalid argument";
        case STPI_EUNSUPPORTED: return "unsupported problem";
        case STPI_EZERO_NORM: return "zero norm (A x = 0)";
        case STPI_ENONFINITE: return "non-finite value";
        case STPI_EHIP: return "HIP runtime error";
        case STPI_EWORKSPACE: return "workspace missing or too small";
        default: return "unknown status";
    }
}

const char *stpi_last_error(void) { return g_last_error.c_str(); }

const char *stpi_version(void) { return "stpi 0.1 gfx950"; }

size_t stpi_workspace_bytes(const stpi_problem *p) {
    if (validate_problem(p) != STPI_OK) return 0;
    return layout_for(p).total;
}

// Matrix-core variants scale their half-precision operands by a bound on
// |f x_stored| (times |x_scale|, applied in the kernel); it is computed here
// into the workspace's state area, which a single step does not otherwise use.
static hipError_t single_step_bound(const Variant *v, const stpi_problem *p, const void *f, const void *x, void *ws,
                                    FwdLaunch &FL, hipStream_t s) {
    if (v->PIPE != 3) return hipSuccess;
    uint32_t *w = &((DevState *)ws)->ubound;
    FL.ubound = w;
    hipError_t e = launch_clear_word(w, s);
    if (e == hipSuccess) e = ops_for(p->dtype)->bound((size_t)p->T * p->H * p->W, f, x, w, s);
    return e;
}

int stpi_step(const stpi_problem *p, const void *f, const void *x, double x_scale, void *z, double *d_sums,
              void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    int rc = validate_problem(p);
    if (rc) return rc;
    if (!f || !x || !z || !d_sums) return fail(STPI_EINVAL, "NULL buffer");
    if (z == f || z == x) return fail(STPI_EINVAL, "z must not alias f or x");
    if (!std::isfinite(x_scale)) return fail(STPI_EINVAL, "x_scale must be finite");
    const WsLayout L = layout_for(p);
    if (!ws || ws_bytes < L.total) return fail(STPI_EWORKSPACE, "workspace needs %zu bytes", L.total);
    const Variant *v = choose_variant(p, forced_variant());
    if (!v) return fail(STPI_EUNSUPPORTED, "no compiled kernel for radii (%d, %d)", p->r_s, p->r_t);
    hipStream_t s = (hipStream_t)stream;
    FwdLaunch FL;
    std::memset(&FL, 0, sizeof(FL));
    FL.f = f;
    FL.buf0 = const_cast<void *>(x);
    FL.buf1 = z;
    FL.state = nullptr;
    FL.x_scale = x_scale;
    FL.partials = (double *)((char *)ws + L.partials_off);
    FL.T = p->T;
    FL.H = p->H;
    FL.W = p->W;
    FL.nseg = segments_for(*v, p);
    make_taps(p, FL.gs, FL.gt);
    hipError_t e = single_step_bound(v, p, f, x, ws, FL, s);
    if (e != hipSuccess) return hip_fail(e, "operand bound");
    e = v->launch(FL, s);
    if (e != hipSuccess) return hip_fail(e, "step kernel launch");
    e = launch_step_sums(FL.partials, grid_blocks(*v, p), x_scale, d_sums, s);
    if (e != hipSuccess) return hip_fail(e, "step sums launch");
    return STPI_OK;
}

}  // extern "C"

namespace stpi {

// Scratch of stpi_step_noalloc: the operand-bound word (first 256 bytes) and
// the step kernel's per-workgroup partial sums. Each device holds its own copy
// for the life of the process; host code reaches it only through the address
// hipGetSymbolAddress returns on that device (the array's name on the host is
// a stand-in, not a device address).
static __device__ __align__(256) unsigned char scratch[STPI_NOALLOC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static void *g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mu;

// The scratch address on the current device (looked up once per device).
static int scratch_for_current_device(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= MAX_DEVICES) return fail(STPI_EUNSUPPORTED, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!ptr) return fail(STPI_EHIP, "hipGetSymbolAddress(scratch) returned NULL");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return STPI_OK;
}

}  // namespace stpi

extern "C" {

size_t stpi_step_noalloc_scratch_bytes(const stpi_problem *p) {
    if (validate_problem(p) != STPI_OK) return 0;
    const Variant *v = choose_variant(p, forced_variant());
    if (!v) return 0;
    return 256 + (size_t)grid_blocks(*v, p) * 2 * sizeof(double);
}

int stpi_step_noalloc(const stpi_problem *p, const void *f, const void *x, double x_scale, void *z, double *d_sums,
                      void *stream) {
    clear_error();
    int rc = validate_problem(p);
    if (rc) return rc;
    if (!f || !x || !z || !d_sums) return fail(STPI_EINVAL, "NULL buffer");
    if (z == f || z == x) return fail(STPI_EINVAL, "z must not alias f or x");
    if (!std::isfinite(x_scale)) return fail(STPI_EINVAL, "x_scale must be finite");
    const Variant *v = choose_variant(p, forced_variant());
    if (!v) return fail(STPI_EUNSUPPORTED, "no compiled kernel for radii (%d, %d)", p->r_s, p->r_t);
    const int nunits = grid_blocks(*v, p);
    const size_t need = 256 + (size_t)nunits * 2 * sizeof(double);
    if (need > (size_t)STPI_NOALLOC_SCRATCH_BYTES)
        return fail(STPI_EUNSUPPORTED, "frame %dx%d needs %zu bytes of step scratch, above the %d-byte limit", p->H,
                    p->W, need, STPI_NOALLOC_SCRATCH_BYTES);
    void *scr = nullptr;
    if ((rc = scratch_for_current_device(&scr)) != STPI_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    FwdLaunch FL;
    std::memset(&FL, 0, sizeof(FL));
    FL.f = f;
    FL.buf0 = const_cast<void *>(x);
    FL.buf1 = z;
    FL.state = nullptr;
    FL.x_scale = x_scale;
    FL.partials = (double *)((char *)scr + 256);
    FL.T = p->T;
    FL.H = p->H;
    FL.W = p->W;
    FL.nseg = segments_for(*v, p);
    make_taps(p, FL.gs, FL.gt);
    hipError_t e = hipSuccess;
    if (v->PIPE == 3) {
        // the bound word is cleared by a kernel and raised by the bound pass
        uint32_t *w = (uint32_t *)scr;
        FL.ubound = w;
        e = launch_clear_word(w, s);
        if (e == hipSuccess) e = ops_for(p->dtype)->bound((size_t)p->T * p->H * p->W, f, x, w, s);
        if (e != hipSuccess) return hip_fail(e, "operand bound");
    }
    e = v->launch(FL, s);
    if (e != hipSuccess) return hip_fail(e, "step kernel launch");
    e = launch_step_sums(FL.partials, nunits, x_scale, d_sums, s);
    if (e != hipSuccess) return hip_fail(e, "step sums launch");
    return STPI_OK;
}

int stpi_iterate(const stpi_problem *p, const void *f, void *x, int init, int max_iters, double tol, void *ws,
                 size_t ws_bytes, stpi_result *out, void *stream) {
    clear_error();
    int rc = validate_problem(p);
    if (rc) return rc;
    if (!f || !x) return fail(STPI_EINVAL, "NULL buffer");
    if (f == x) return fail(STPI_EINVAL, "x must not alias f");
    if (max_iters < 0) return fail(STPI_EINVAL, "max_iters must be >= 0");
    if (init < 0 || init > 2) return fail(STPI_EINVAL, "init must be 0 (use x), 1 (uniform) or 2 (use x, rise check)");
    if (!std::isfinite(tol)) return fail(STPI_EINVAL, "tol must be finite");
    const WsLayout L = layout_for(p);
    if (!ws || ws_bytes < L.total) return fail(STPI_EWORKSPACE, "workspace needs %zu bytes", L.total);
    const Variant *v = choose_variant(p, forced_variant());
    if (!v) return fail(STPI_EUNSUPPORTED, "no compiled kernel for radii (%d, %d)", p->r_s, p->r_t);
    if (out) std::memset(out, 0, sizeof(*out));
    hipStream_t s = (hipStream_t)stream;
    const DtypeOps *ops = ops_for(p->dtype);
    const size_t N = (size_t)p->T * p->H * p->W;
    const ChainMem m = chain_mem(L, ws);

    // A run in tolerance mode stops early, but a chain of max_iters steps
    // would still launch every (step, finalise) pair (they exit at once when
    // done, at a launch latency each). Long tolerance runs therefore replay a
    // chain of CHAIN_CHUNK steps, the host checking the stop flag one chunk
    // behind so the device never waits for it.
    const bool chunked = tol > 0.0 && max_iters > 2 * CHAIN_CHUNK;
    const int pform = chain_pform(v, max_iters);
    const int defer = chain_defer(v, p);
    ChainArgs ca{p, ops, v, f, x, m, init, max_iters, tol, pform, defer};
    const bool use_graphs = s != nullptr && graphs_enabled();
    auto run = [&](int part) -> int {
        if (!use_graphs) return enqueue_chain_part(ca, part, s);
        GraphKey key;
        std::memset(&key, 0, sizeof(key));
        key.p = *p;
        key.f = f;
        key.x = x;
        key.ws = ws;
        key.init = init;
        key.max_iters = max_iters;
        key.tol = tol;
        key.v = v;
        key.s = s;
        key.part = part;
        key.pform = pform;
        key.defer = defer;
        return launch_cached_graph(key, [&] { return enqueue_chain_part(ca, part, s); }, s);
    };
    if (!chunked) {
        if ((rc = run(CHAIN_ALL))) return rc;
    } else {
        if ((rc = run(CHAIN_HEAD))) return rc;
        DevState *poll = pinned_state();
        hipEvent_t ev = poll_event();
        if (!poll || !ev) return fail(STPI_EHIP, "pinned poll buffer or event unavailable");
        hipError_t e;
        for (int issued = CHAIN_CHUNK; issued < max_iters; issued += CHAIN_CHUNK) {
            // state after the chunks issued so far (their last step not yet
            // finalised), then one more chunk while it travels
            if ((e = hipMemcpyAsync(poll, m.state, sizeof(DevState), hipMemcpyDeviceToHost, s)) != hipSuccess)
                return hip_fail(e, "state poll");
            if ((e = hipEventRecord(ev, s)) != hipSuccess) return hip_fail(e, "poll event");
            if ((rc = run(CHAIN_CHUNK_PART))) return rc;
            if ((e = hipEventSynchronize(ev)) != hipSuccess) return hip_fail(e, "poll wait");
            if (poll->done) break;
        }
        if ((rc = run(CHAIN_TAIL))) return rc;
    }
    if (!out) return STPI_OK;

    DevState hs;
    hipError_t e = hipMemcpyAsync(&hs, m.slot(FINAL_SLOT), sizeof(hs), hipMemcpyDeviceToHost, s);
    if (e != hipSuccess) return hip_fail(e, "state readback");
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "stream synchronize");
    out->iters = hs.iters;
    out->converged = hs.converged;
    out->flags = hs.flags;
    out->residual = hs.residual;
    out->lambda = hs.lambda;
    out->rayleigh = hs.rayleigh;
    out->first_residuals[0] = hs.first_res[0];
    out->first_residuals[1] = hs.first_res[1];
    out->status = STPI_OK;
    if (hs.flags & FLAG_NONFINITE) out->status = STPI_ENONFINITE;
    else if (hs.flags & FLAG_ZERO) out->status = STPI_EZERO_NORM;
    (void)N;
    if (out->status != STPI_OK)
        return fail(out->status, "iteration stopped after %d steps: %s", hs.iters, stpi_status_string(out->status));
    return STPI_OK;
}

int stpi_time_step(const stpi_problem *p, const void *f, const void *x, void *z, void *ws, size_t ws_bytes,
                   int variant, int reps, void *stream, double *avg_ms) {
    clear_error();
    int rc = validate_problem(p);
    if (rc) return rc;
    if (!f || !x || !z || !avg_ms) return fail(STPI_EINVAL, "NULL buffer");
    if (reps < 1) return fail(STPI_EINVAL, "reps must be >= 1");
    const WsLayout L = layout_for(p);
    if (!ws || ws_bytes < L.total) return fail(STPI_EWORKSPACE, "workspace needs %zu bytes", L.total);
    const Variant *v = choose_variant(p, variant >= 0 ? variant : forced_variant());
    if (!v) return fail(STPI_EUNSUPPORTED, "no eligible kernel variant");
    hipStream_t s = (hipStream_t)stream;
    FwdLaunch FL;
    std::memset(&FL, 0, sizeof(FL));
    FL.f = f;
    FL.buf0 = const_cast<void *>(x);
    FL.buf1 = z;
    FL.x_scale = 1.0;
    FL.partials = (double *)((char *)ws + L.partials_off);
    FL.T = p->T;
    FL.H = p->H;
    FL.W = p->W;
    FL.nseg = segments_for(*v, p);
    make_taps(p, FL.gs, FL.gt);
    hipEvent_t e0, e1;
    hipError_t e;
    if ((e = single_step_bound(v, p, f, x, ws, FL, s)) != hipSuccess) return hip_fail(e, "operand bound");
    if ((e = hipEventCreate(&e0)) != hipSuccess) return hip_fail(e, "event create");
    if ((e = hipEventCreate(&e1)) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return hip_fail(e, "event create");
    }
    e = hipEventRecord(e0, s);
    for (int i = 0; i < reps && e == hipSuccess; ++i) e = v->launch(FL, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return hip_fail(e, "timed launches");
    *avg_ms = (double)ms / reps;
    return STPI_OK;
}

int stpi_time_chain_step(const stpi_problem *p, const void *f, void *x, void *ws, size_t ws_bytes, int variant,
                         int reps, void *stream, double *avg_ms, int *product_form) {
    clear_error();
    int rc = validate_problem(p);
    if (rc) return rc;
    if (!f || !x || !avg_ms) return fail(STPI_EINVAL, "NULL buffer");
    if (f == x) return fail(STPI_EINVAL, "x must not alias f");
    if (reps < 1) return fail(STPI_EINVAL, "reps must be >= 1");
    const WsLayout L = layout_for(p);
    if (!ws || ws_bytes < L.total) return fail(STPI_EWORKSPACE, "workspace needs %zu bytes", L.total);
    const Variant *v = choose_variant(p, variant >= 0 ? variant : forced_variant());
    if (!v) return fail(STPI_EUNSUPPORTED, "no eligible kernel variant");
    hipStream_t s = (hipStream_t)stream;
    const DtypeOps *ops = ops_for(p->dtype);
    const ChainMem m = chain_mem(L, ws);
    // a fixed-count chain long enough that no timed step finds it done
    const int total = reps + 2;
    const int pform = chain_pform(v, total);
    const int defer = chain_defer(v, p);
    if (product_form) *product_form = pform;
    rc = enqueue_chain_init(p, ops, x, m, 1, total, 0.0, s, v, f, pform);
    // the steps as a fixed-count chain of `total` steps runs them
    if (!rc) rc = enqueue_chain_steps(p, v, f, x, m, 1, s, pform, defer, total, 0);
    if (rc) return rc;
    hipEvent_t e0, e1;
    hipError_t e;
    if ((e = hipEventCreate(&e0)) != hipSuccess) return hip_fail(e, "event create");
    if ((e = hipEventCreate(&e1)) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return hip_fail(e, "event create");
    }
    e = hipEventRecord(e0, s);
    if (e == hipSuccess) rc = enqueue_chain_steps(p, v, f, x, m, reps, s, pform, defer, total, 1);
    if (e == hipSuccess && !rc) e = hipEventRecord(e1, s);
    if (e == hipSuccess && !rc) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess && !rc) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    if (e != hipSuccess) return hip_fail(e, "timed launches");
    *avg_ms = (double)ms / reps;
    return STPI_OK;
}

int stpi_variant_count(int dtype) {
    const DtypeOps *ops = ops_for(dtype);
    return ops ? ops->nvariants : 0;
}

int stpi_variant_info(int dtype, int index, int32_t info[9]) {
    clear_error();
    const DtypeOps *ops = ops_for(dtype);
    if (!ops || !info || index < 0 || index >= ops->nvariants)
        return fail(STPI_EINVAL, "no variant %d for dtype %d", index, dtype);
    const Variant &v = ops->variants[index];
    info[0] = v.RS;
    info[1] = v.RT;
    info[2] = v.TH;
    info[3] = v.TW;
    info[4] = v.NTHR;
    info[5] = v.RY;
    info[6] = v.QX;
    info[7] = v.OCC;
    info[8] = v.PIPE;
    return STPI_OK;
}

int stpi_launch_shape(const stpi_problem *p, int variant, int32_t info[5]) {
    clear_error();
    int rc = validate_problem(p);
    if (rc) return rc;
    if (!info) return fail(STPI_EINVAL, "NULL info");
    const DtypeOps *ops = ops_for(p->dtype);
    const Variant *v = choose_variant(p, variant >= 0 ? variant : forced_variant());
    if (!v) return fail(STPI_EUNSUPPORTED, "no compiled kernel for radii (%d, %d)", p->r_s, p->r_t);
    const int nseg = segments_for(*v, p);
    info[0] = (int32_t)(v - ops->variants);
    info[1] = grid_blocks(*v, p) / nseg;
    info[2] = nseg;
    info[3] = v->blocks_per_cu();
    info[4] = grid_blocks(*v, p);
    return STPI_OK;
}

int stpi_set_variant(int index) {
    clear_error();
    if (index < -1) return fail(STPI_EINVAL, "variant index must be >= -1");
    set_forced_variant(index);
    return STPI_OK;
}

}  // extern "C"

namespace stpi {

int chain_defer(const Variant *v, const stpi_problem *p) {
    return grid_blocks(*v, p) <= DEFER_MAX_UNITS && !fusion_disabled() ? 1 : 0;
}

// Enqueues start vector, max_iters steps and the final pass. No host
// synchronisation.
int enqueue_chain_init(const stpi_problem *p, const DtypeOps *ops, void *x, const ChainMem &m, int init,
                       int max_iters, double tol, hipStream_t s, const Variant *v, const void *f, int pform) {
    const size_t N = (size_t)p->T * p->H * p->W;
    DevState *state = m.state;
    hipError_t e;
    if (init == 1) {
        // product form: the first step stages f itself, the constant start is never stored
        e = pform ? launch_state_init(state, 1.0 / std::sqrt((double)N), tol, max_iters, 0, 2, s)
                  : ops->uniform_start(x, N, state, tol, max_iters, s);
        if (e != hipSuccess) return hip_fail(e, "init");
    } else {
        if ((e = launch_state_init(state, 1.0, tol, max_iters, init == 2 ? 1 : 0, 0, s)) != hipSuccess)
            return hip_fail(e, "init");
        if ((e = ops->sumsq(x, N, m.partials, s)) != hipSuccess) return hip_fail(e, "norm");
        if ((e = launch_state_from_norm(m.partials, NORM_BLOCKS_HOST, state, s)) != hipSuccess)
            return hip_fail(e, "init norm");
    }
    // matrix-core steps scale their operands by max |f| (the iterate is unit)
    if (v && v->PIPE == 3 && (e = ops->bound(N, f, nullptr, &state->ubound, s)) != hipSuccess)
        return hip_fail(e, "operand bound");
    if (pform && init != 1 && (e = ops->to_product(f, x, m.buf1, N, state, s)) != hipSuccess)
        return hip_fail(e, "product-form start");
    return STPI_OK;
}

int enqueue_chain_tail(const stpi_problem *p, const DtypeOps *ops, const Variant *v, const void *f, void *x,
                       const ChainMem &m, int steps, hipStream_t s, int pform, int defer) {
    const size_t N = (size_t)p->T * p->H * p->W;
    if (steps <= 0) defer = 0;
    const DevState *last = m.slot(defer ? steps & 1 : 0);
    StepPartials part = m.set((steps + 1) & 1);
    if (!pform) part.wmax = nullptr;
    const int np = defer ? grid_blocks(*v, p) : 0;
    const hipError_t e = pform ? ops->from_product(x, m.buf1, f, N, last, part, np, m.slot(FINAL_SLOT), s)
                               : ops->normalize(x, m.buf1, N, last, part, np, m.slot(FINAL_SLOT), s);
    return e == hipSuccess ? STPI_OK : hip_fail(e, "normalize");
}

int enqueue_chain_steps(const stpi_problem *p, const Variant *v, const void *f, void *x, const ChainMem &m, int steps,
                        hipStream_t s, int pform, int defer, int fixed_total, int k0) {
    hipError_t e;
    FwdLaunch FL;
    std::memset(&FL, 0, sizeof(FL));
    FL.f = f;
    FL.buf0 = x;
    FL.buf1 = m.buf1;
    FL.T = p->T;
    FL.H = p->H;
    FL.W = p->W;
    FL.nseg = segments_for(*v, p);
    FL.ubound = &m.state->ubound;
    make_taps(p, FL.gs, FL.gt);
    const int nb = grid_blocks(*v, p);
    const FwdLaunchFn launch = pform ? v->launch_p : v->launch;
    if (!launch) return fail(STPI_EUNSUPPORTED, "variant has no product-form step");
    for (int k = 0; k < steps; ++k) {
        const int kk = k0 + k, slot = defer ? kk & 1 : 0;
        FL.no_prev = fixed_total > 0 && kk >= 2 && kk < fixed_total - 1 ? 1 : 0;
        FL.state = m.slot(slot);
        FL.state_out = defer ? m.slot(slot ^ 1) : nullptr;
        const StepPartials mine = m.set(slot);
        FL.partials = mine.sums;
        FL.wpart = mine.wmax;
        FL.prev_part = m.set(slot ^ 1);
        if ((e = launch(FL, s)) != hipSuccess) return hip_fail(e, "step kernel launch");
        if (!defer) {
            StepPartials part = mine;
            if (!pform) part.wmax = nullptr;
            if ((e = launch_finalize(part, nb, m.state, s)) != hipSuccess) return hip_fail(e, "finalize launch");
        }
    }
    return STPI_OK;
}

int enqueue_iteration(const stpi_problem *p, const DtypeOps *ops, const Variant *v, const void *f, void *x,
                      const ChainMem &m, int init, int max_iters, double tol, hipStream_t s, int pform, int defer) {
    int rc = enqueue_chain_init(p, ops, x, m, init, max_iters, tol, s, v, f, pform);
    if (!rc) rc = enqueue_chain_steps(p, v, f, x, m, max_iters, s, pform, defer, tol > 0.0 ? 0 : max_iters);
    return rc ? rc : enqueue_chain_tail(p, ops, v, f, x, m, max_iters, s, pform, defer);
}

}  // namespace stpi
