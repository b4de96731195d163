// Host side of the pair path (bc_pair.hip): which graphs take it, its
// workspaces and its level loop.
#include "bc_runtime.h"

namespace bcx {

// Scratch of one call: the sources that fit run together.
constexpr size_t kPairBudget = (size_t)4 << 30;

// Undirected graphs of low degree: a lane takes a vertex's arcs one after
// another, and road-like networks have few of them.
bool pair_fits(const bc_graph_s *g) {
    return !g->directed && g->n > 0 && g->n < (1 << 28) && g->max_deg <= kPairMaxDeg &&
           g->nnz <= 8 * (int64_t)g->n;
}

// ... that are deep (see kPairDepth).
bool use_pair(const bc_graph_s *g, int32_t level_loop, int32_t width) {
    return level_loop == BC_LOOP_AUTO && width <= kWave && pair_fits(g) && g->deep;
}

static size_t pair_stride(const bc_graph_s *g) { return ((size_t)g->n + 15) & ~(size_t)15; }

// How a call is run: the kind of level loop, the levels its arrays hold, and
// whether counts carry exponents.
struct PairShape {
    bool solo = false;  // one workgroup per source, else a launch per level
    bool ext = false;
    int32_t lcap = 0;
};

// Bytes per source.
static size_t pair_source_bytes(const bc_graph_s *g, const PairShape &sh) {
    const size_t cell = sizeof(int32_t) + 2 * sizeof(double) +
                        (sh.solo ? sizeof(double) : sizeof(uint8_t)) +
                        (sh.ext ? sizeof(int32_t) : 0);
    return pair_stride(g) * cell + (size_t)sh.lcap * 2 * sizeof(int32_t) + 3 * sizeof(int32_t);
}

static size_t pair_ws_bytes(const bc_graph_s *g, int32_t k, const PairShape &sh) {
    return (size_t)k * pair_source_bytes(g, sh) + 12 * kAlign;
}

static PairShape pair_shape(const bc_graph_s *g, int32_t k) {
    PairShape sh;
    sh.ext = g->pair_ext.load() || g->sigma_ext.load();
    sh.lcap = std::max(1024, g->pair_depth_hint.load() + 64);
    // Estimated times, fitted to road-like grids of 90K to 1M vertices, 90 to
    // 1,700 levels and 1 to 256 sources (MI355X).  A launch per level: 11 us
    // per level (both passes) and 0.18 ns per pair.  A workgroup per source:
    // 2.75 us per level, and 8.2 ns per pair of a source on its one compute
    // unit, 0.23 ns per pair over the device.  For instance, in ms, launches
    // against workgroups: 1024^2 with shortcuts (122 levels), 1 source 1.9 /
    // 9.0, 64 sources 12.2 / 15.7; without shortcuts (1,700 levels), 64
    // sources 31.6 / 18.7; 300^2 with shortcuts, 64 sources 2.2 / 1.1.
    const double n = (double)g->n, pairs = n * (double)k;
    const int32_t hint = g->pair_depth_hint.load();
    const double levels = hint > 0 ? (double)hint : g->depth_guess;
    const double launches = 0.5e-3 + levels * 11e-6 + pairs * 0.18e-9;
    const double alone = levels * 2.75e-6 +
                         std::max(n * 8.2e-9 * std::ceil((double)k / kCus), pairs * 0.23e-9);
    sh.solo = deep_lds_bytes(g->n) <= kSrcLdsBytes && alone < launches;
    return sh;
}

// Sources run together of a call of k: whole groups of those that pair_sum
// adds together, so that a call's sums are the same however many rounds its
// shape (which follows the depth seen) makes of it.  The budget is rounded up
// to such a group (at most seven sources more): rounded down, a call of a few
// sources past the last group paid for a second round's levels (ms, grids with
// shortcuts: 1M vertices, 193 sources 38.3, so 36.3; 4M, 49 sources 38.2, 36.3).
static int32_t pair_cap(const bc_graph_s *g, int32_t k, const PairShape &sh) {
    const int64_t fit = (int64_t)(kPairBudget / pair_source_bytes(g, sh));
    const int64_t room = std::max<int64_t>((fit + kPairSum - 1) / kPairSum, 1) * kPairSum;
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(k, room));
}

// Bytes of the vertex order: the rows pos, row_ptr and caller, the first arcs
// and the ids; and of the scratch rows that building it takes besides.
static size_t layout_row(const bc_graph_s *g) {
    return align_up(((size_t)g->n + 1) * sizeof(int32_t));
}
static size_t layout_bytes(const bc_graph_s *g) {
    return 3 * layout_row(g) + align_up((size_t)g->n * sizeof(int4)) +
           align_up((size_t)std::max<int64_t>(g->nnz, 1) * sizeof(int32_t));
}
constexpr int kLayoutScratch = 6;

size_t pair_bytes(const bc_graph_s *g, int32_t k) {
    const PairShape sh = pair_shape(g, std::max(k, 1));
    return layout_bytes(g) + std::max(pair_ws_bytes(g, pair_cap(g, std::max(k, 1), sh), sh),
                                      kLayoutScratch * layout_row(g));
}

size_t layout_held(bc_graph_s *g) {
    std::lock_guard<std::mutex> lk(g->layout_mu);
    return g->layout.bytes;
}

void layout_trim(bc_graph_s *g) {
    std::lock_guard<std::mutex> lk(g->layout_mu);
    if (!g->layout.block || g->layout.users > 0) return;
    (void)hipFree(g->layout.block);
    g->layout = bc_graph_s::Layout{};
}

void pair_ws_destroy(PairWS *ws) {
    if (!ws) return;
    ws->timer.destroy();
    if (ws->d_stats) (void)hipFree(ws->d_stats);
    if (ws->block) (void)hipFree(ws->block);
    if (ws->h_depth) (void)hipHostFree(ws->h_depth);
    delete ws;
}

// Memory of `ws` for k sources, cut up.
static bc_status pair_room(bc_graph_s *g, PairWS *ws, int32_t k, const PairShape &sh) {
    const size_t need = pair_ws_bytes(g, k, sh);
    if (ws->bytes < need) {
        auto set_bytes = [&](size_t b) {  // (bc_workspace_held reads it)
            std::lock_guard<std::mutex> lk(g->mu);
            ws->bytes = b;
        };
        if (ws->block) (void)hipFree(ws->block);
        ws->block = nullptr;
        set_bytes(0);
        BC_TRY_HIP(hipMalloc(&ws->block, need));
        set_bytes(need);
    }
    if (ws->depth_cap < k + 1) {
        if (ws->h_depth) (void)hipHostFree(ws->h_depth);
        ws->h_depth = nullptr;
        ws->depth_cap = 0;
        BC_TRY_HIP(hipHostMalloc((void **)&ws->h_depth, 2 * ((size_t)k + 1) * sizeof(int32_t),
                                 hipHostMallocDefault));
        ws->depth_cap = k + 1;
    }
    char *p = (char *)ws->block;
    auto take = [&](size_t b) {
        char *r = p;
        p += align_up(b);
        return (void *)r;
    };
    PairDev &d = ws->dev;
    d = PairDev{};
    d.n = g->n;
    d.k = k;
    d.lcap = sh.lcap;
    d.stride = pair_stride(g);
    d.g = {g->layout.row_ptr, g->layout.col_idx, g->layout.four};
    d.pos = g->layout.pos;
    const size_t cells = (size_t)k * d.stride;
    d.val = (double *)take(cells * sizeof(double));
    d.delta = (double *)take(cells * sizeof(double));
    d.q = (int32_t *)take(cells * sizeof(int32_t));
    if (sh.ext) d.ex = (int32_t *)take(cells * sizeof(int32_t));
    if (sh.solo) d.sig = (double *)take(cells * sizeof(double));
    else d.code = (uint8_t *)take(cells);
    d.cnt = (int32_t *)take((size_t)sh.lcap * k * sizeof(int32_t));
    d.lvl = (int32_t *)take((size_t)sh.lcap * k * sizeof(int32_t));
    // the depths and, behind them, the range flag: read back together
    d.depth = (int32_t *)take(((size_t)k + 1) * sizeof(int32_t));
    d.range = d.depth + k;
    d.src = (int32_t *)take((size_t)k * sizeof(int32_t));
    d.at = (int32_t *)take((size_t)k * sizeof(int32_t));
    return BC_OK;
}

// An idle workspace of the graph (calls return with their work finished), or
// a new one.
static bc_status pair_acquire(bc_graph_s *g, PairWS **out) {
    PairWS *ws = nullptr;
    {
        std::lock_guard<std::mutex> lk(g->mu);
        for (PairWS *w : g->pair_pool)
            if (!w->busy && (!ws || w->bytes > ws->bytes)) ws = w;
        if (ws) ws->busy = true;
    }
    if (!ws) {
        ws = new (std::nothrow) PairWS();
        if (!ws) return BC_ERR_OUT_OF_MEMORY;
        ws->busy = true;
        std::lock_guard<std::mutex> lk(g->mu);
        g->pair_pool.push_back(ws);
    }
    *out = ws;
    return BC_OK;
}

// The graph's pair-path vertex order, built on first use, for one more run
// (BC_OK: until layout_release).
static bc_status layout_acquire(bc_graph_s *g, hipStream_t stream) {
    std::lock_guard<std::mutex> lk(g->layout_mu);
    auto &l = g->layout;
    if (l.block) {
        ++l.users;
        return BC_OK;
    }
    const size_t row = layout_row(g);
    const size_t quad = align_up((size_t)g->n * sizeof(int4));
    void *block = nullptr, *tmp = nullptr;
    hipError_t e = hipMalloc(&block, layout_bytes(g));
    if (e == hipSuccess) e = hipMalloc(&tmp, kLayoutScratch * row);
    if (e == hipSuccess) {
        l.pos = (int32_t *)block;
        l.row_ptr = (int32_t *)((char *)block + row);
        l.caller = (int32_t *)((char *)block + 2 * row);
        l.four = (int4 *)((char *)block + 3 * row);
        l.col_idx = (int32_t *)((char *)block + 3 * row + quad);
        LayoutDev d{};
        d.n = g->n;
        d.row_ptr = g->d_row_ptr;
        d.col_idx = g->d_col_idx;
        d.iperm = g->d_iperm;
        for (int i = 0; i < kLayoutScratch; ++i) d.tmp[i] = (int32_t *)((char *)tmp + (size_t)i * row);
        d.pos = l.pos;
        d.new_rp = l.row_ptr;
        d.new_col = l.col_idx;
        d.caller = l.caller;
        d.four = l.four;
        e = layout_build(d, stream);
        const hipError_t es = hipStreamSynchronize(stream);
        if (e == hipSuccess) e = es;
    }
    if (tmp) (void)hipFree(tmp);
    if (e != hipSuccess) {
        if (block) (void)hipFree(block);
        l = bc_graph_s::Layout{};
        return from_hip(e);
    }
    l.block = block;
    l.bytes = layout_bytes(g);
    l.users = 1;
    return BC_OK;
}

static void layout_release(bc_graph_s *g) {
    std::lock_guard<std::mutex> lk(g->layout_mu);
    --g->layout.users;
}

// How a round of sources ended: done, with a count past double's range, or
// with more levels than the arrays hold.
enum class PairEnd { Done, Range, Grow };

// A round of m sources, a launch per level; the sources are in d.src.
static hipError_t level_round(bc_graph_s *g, PairWS *ws, int32_t m, hipStream_t stream, bool prof,
                              int32_t &deepest, PairEnd &end) {
    PairDev &d = ws->dev;
    const int32_t period = std::max(1, g->profiling.load());
    auto measure = [&](int32_t L) {
        ws->timer.on = prof && L % period == 0;
        d.stats = ws->timer.on ? ws->d_stats : nullptr;
    };
    hipError_t e = pair_start(d, stream);
    // workgroups per source: the launches' 256-pair pieces at the average
    // level width of the last run, twice over, within the device's room
    const int32_t hint = g->pair_depth_hint.load();
    const int64_t width = 2 * ((int64_t)g->n / (std::max(hint, 64) + 1) / kBlock + 1);
    const int32_t per =
        (int32_t)std::max<int64_t>(1, std::min<int64_t>(width, std::max(1, kMaxGridBlocks / m)));
    for (int32_t L0 = 0; e == hipSuccess;) {
        // the levels of the last run and one more in one chunk, then 64 at a
        // time; a level past the deepest finds empty queues
        const int32_t K = L0 == 0 && hint > 0 ? hint + 2 : 64;
        const int32_t Lend = std::min(L0 + K, d.lcap - 1);
        for (int32_t L = L0; L < Lend && e == hipSuccess; ++L) {
            measure(L);
            e = ws->timer.begin(BC_PROF_FORWARD, stream);
            if (e == hipSuccess) e = pair_forward(d, L, per, stream);
            if (e == hipSuccess) e = ws->timer.end(stream);
        }
        if (e == hipSuccess)
            e = hipMemcpyAsync(ws->h_depth, d.depth, ((size_t)m + 1) * sizeof(int32_t),
                               hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return e;
        deepest = *std::max_element(ws->h_depth, ws->h_depth + m);
        if (ws->h_depth[m]) {
            end = PairEnd::Range;
            return hipSuccess;
        }
        if (deepest < Lend - 1) break;  // level Lend-1 was empty
        if (Lend >= d.lcap - 1) {       // no room for the next level
            end = PairEnd::Grow;
            return hipSuccess;
        }
        L0 = Lend;
    }
    for (int32_t L = deepest; L >= 1 && e == hipSuccess; --L) {
        measure(L);
        e = ws->timer.begin(BC_PROF_REVERSE, stream);
        if (e == hipSuccess) e = pair_reverse(d, L, per, stream);
        if (e == hipSuccess) e = ws->timer.end(stream);
    }
    return e;
}

// A round of m sources, a workgroup each: two launches.
static hipError_t solo_round(bc_graph_s *g, PairWS *ws, int32_t m, hipStream_t stream, bool prof,
                             int32_t &deepest, PairEnd &end) {
    (void)g;
    PairDev &d = ws->dev;
    ws->timer.on = prof;
    d.stats = prof ? ws->d_stats : nullptr;
    hipError_t e = deep_source(d, 0, stream);
    if (e == hipSuccess) e = ws->timer.begin(BC_PROF_FORWARD, stream);
    if (e == hipSuccess) e = deep_source(d, 1, stream);
    if (e == hipSuccess) e = ws->timer.end(stream);
    // (queued before the depths are known: harmless where the round is run again)
    if (e == hipSuccess) e = ws->timer.begin(BC_PROF_REVERSE, stream);
    if (e == hipSuccess) e = deep_source(d, 2, stream);
    if (e == hipSuccess) e = ws->timer.end(stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws->h_depth, d.depth, ((size_t)m + 1) * sizeof(int32_t),
                           hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return e;
    deepest = *std::max_element(ws->h_depth, ws->h_depth + m);
    if (ws->h_depth[m]) end = PairEnd::Range;
    else if (*std::min_element(ws->h_depth, ws->h_depth + m) < 0) end = PairEnd::Grow;
    return hipSuccess;
}

// All sources, as many at a time as the budget and the free memory hold, each
// round's dependencies added to bc_out (caller order) in source order.
// Returns with all work finished; BC_ERR_OUT_OF_MEMORY where not even one
// source at a time fits.
bc_status pair_run(bc_graph_s *g, const int32_t *sources, int32_t k, double *bc_out,
                   hipStream_t stream) {
    const bc_status sl = layout_acquire(g, stream);
    if (sl != BC_OK) return sl;
    PairShape sh = pair_shape(g, k);
    int32_t most = std::max(k, 1);  // sources of a round that memory has room for
    PairWS *ws = nullptr;
    bc_status st = pair_acquire(g, &ws);
    struct Held {
        bc_graph_s *g;
        PairWS *&ws;
        ~Held() {
            layout_release(g);
            if (!ws) return;
            std::lock_guard<std::mutex> lk(g->mu);
            ws->busy = false;
        }
    } held{g, ws};
    if (st != BC_OK) return st;
    const bool prof = g->profiling.load() != 0;
    ws->timer.on = false;
    ws->timer.used = 0;
    hipError_t e = hipSuccess;
    // the counters of every round of the call, those run again included (not in
    // the block, which each round cuts anew)
    if (prof) {
        if (!ws->d_stats)
            BC_TRY_HIP(hipMalloc(&ws->d_stats, kStatWords * sizeof(unsigned long long)));
        BC_TRY_HIP(hipMemsetAsync(ws->d_stats, 0, kStatWords * sizeof(unsigned long long), stream));
    }
    int32_t run_depth = 0;
    int64_t level_steps = 0;
    for (int32_t s0 = 0; s0 < k;) {
        const int32_t m = std::min({pair_cap(g, k, sh), most, k - s0});
        st = pair_room(g, ws, m, sh);
        if (st == BC_ERR_OUT_OF_MEMORY && m > 1) {
            (void)hipGetLastError();  // (or the next launch would report it)
            most = m > kPairSum ? (m / 2 + kPairSum - 1) / kPairSum * kPairSum : m / 2;
            most = std::min(most, m - 1);
            continue;
        }
        if (st != BC_OK) return st;
        PairDev &d = ws->dev;
        int32_t *h_src = ws->h_depth + m + 1;
        for (int32_t i = 0; i < m; ++i) h_src[i] = g->h_perm[(size_t)sources[s0 + i]];
        e = hipMemcpyAsync((void *)d.src, h_src, (size_t)m * sizeof(int32_t), hipMemcpyHostToDevice,
                           stream);
        int32_t deepest = 0;
        PairEnd end = PairEnd::Done;
        if (e == hipSuccess)
            e = sh.solo ? solo_round(g, ws, m, stream, prof, deepest, end)
                        : level_round(g, ws, m, stream, prof, deepest, end);
        if (e == hipSuccess && end == PairEnd::Done)
            e = pair_sum(d, g->layout.caller, bc_out, s0 > 0, stream);
        // (the source table is rewritten by the next round)
        const hipError_t es = hipStreamSynchronize(stream);
        if (e == hipSuccess) e = es;
        if (e != hipSuccess) return from_hip(e);
        if (end == PairEnd::Range) {  // these sources again with exponents
            g->pair_ext.store(true);
            sh.ext = true;
            continue;
        }
        if (end == PairEnd::Grow) {  // with room for more levels
            sh.lcap = (int32_t)std::min<int64_t>((int64_t)sh.lcap * 2, (int64_t)g->n + 2);
            continue;
        }
        for (int32_t i = 0; i < m; ++i) level_steps += 2 * (int64_t)ws->h_depth[i] + 1;
        run_depth = std::max(run_depth, deepest);
        s0 += m;
    }
    if (k == 0) {
        e = hipMemsetAsync(bc_out, 0, (size_t)g->n * sizeof(double), stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        return from_hip(e);
    }
    g->pair_depth_hint.store(run_depth);
    if (prof) accumulate_profile(g, ws->timer, ws->d_stats, level_steps);
    return BC_OK;
}

}  // namespace bcx
