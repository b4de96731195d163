// Host side of the one-workgroup-per-source path (bc_source.hip): which calls
// take it, the split of a call's requests into units (one workgroup each),
// and the workspaces of a launch.
#include "bc_runtime.h"

namespace bcx {

// A launch's scratch per graph is kept under this, or under what every unit the
// device runs at once takes (where values are in LDS 0.7 MB each for the largest
// graph, 256 at a time; up to 4.7 MB where they are not); longer calls take
// several launches.  A request's units (at most those) go in one launch.
constexpr size_t kSourceBudget = (size_t)512 << 20;

// Largest graph that this path takes with the values in memory: beyond it the
// host loop was faster on every measured shape (see source_seconds).
constexpr int32_t kSrcMemN = 1 << 17;

// A source's values fit LDS, or memory may hold them, and arc offsets in bytes
// fit 32 bits.
bool source_fits(const bc_graph_s *g) {
    return (source_in_lds(g->n) || g->n <= kSrcMemN) && g->nnz < ((int64_t)1 << 30);
}

// Workgroups of the graph a compute unit holds at once (by LDS; two of 16
// waves are all its wave slots).  With the values in memory one, where arcs are
// many: two run each other's lines out of the L2 (16,384 sources, 21K vertices
// of 16 arcs each: 92 ms with two, 73 with one; of 4 each 24 and 27).
int32_t source_per_cu(const bc_graph_s *g) {
    if (!source_in_lds(g->n) && g->nnz > 8 * (int64_t)g->n) return 1;
    return source_lds_bytes(g->n) * 2 <= kSrcLdsBytes ? 2 : 1;
}

// Sources per unit of a request of k: one while the request's units fit the
// device at once, else enough that they do.  Depends on the request and the
// graph alone, so a request's sums are the same whatever shares its launch.
int32_t source_unit(const bc_graph_s *g, int32_t k) {
    const int32_t room = kCus * source_per_cu(g);
    return std::max(1, (k + room - 1) / room);
}

// Scratch of one unit: its BC row, queue, sigmas and level records.
size_t source_unit_bytes(const bc_graph_s *g) {
    const size_t n = (size_t)std::max<int32_t>(g->n, 1);
    static_assert(kAlign == 32 * sizeof(double), "source_val rounds up to kAlign bytes");
    return 2 * align_up(n * sizeof(double)) + align_up(n * sizeof(int32_t)) +
           align_up((n + 2) * kSrcClasses * sizeof(uint32_t)) +
           (source_in_lds(g->n) ? 0 : align_up((n + 1) * sizeof(double)));
}

// Units a launch runs of a call of `units` (a request's go in one launch).
int32_t source_cap(const bc_graph_s *g, int64_t units) {
    const int64_t fit = std::max<int64_t>((int64_t)(kSourceBudget / source_unit_bytes(g)),
                                          kCus * source_per_cu(g));
    return (int32_t)std::max<int64_t>(1, std::min<int64_t>(std::max<int64_t>(units, 1), fit));
}

void source_ws_destroy(SourceWS *ws) {
    if (!ws) return;
    if (ws->block) (void)hipFree(ws->block);
    if (ws->d_stats) (void)hipFree(ws->d_stats);
    if (ws->h_tab) (void)hipHostFree(ws->h_tab);
    delete ws;
}

// An idle workspace of the graph with room for `cap` units (grown if none is
// large enough), or a new one.  Calls return with their work finished, so a
// released workspace has no reader left.
bc_status source_acquire(bc_graph_s *g, int32_t cap, SourceWS **out) {
    SourceWS *ws = nullptr;
    {
        std::lock_guard<std::mutex> lk(g->mu);
        for (SourceWS *w : g->source_pool)
            if (!w->busy && (!ws || (ws->cap < cap && w->cap > ws->cap))) ws = w;
        if (ws) ws->busy = true;
    }
    if (!ws) {
        ws = new (std::nothrow) SourceWS();
        if (!ws) return BC_ERR_OUT_OF_MEMORY;
        ws->busy = true;
        std::lock_guard<std::mutex> lk(g->mu);
        g->source_pool.push_back(ws);
    }
    *out = ws;
    if (ws->cap >= cap) return BC_OK;
    if (ws->block) (void)hipFree(ws->block);
    ws->block = nullptr;
    ws->bytes = 0;
    ws->cap = 0;
    const size_t bytes = (size_t)cap * source_unit_bytes(g);
    const hipError_t e = hipMalloc(&ws->block, bytes);
    std::lock_guard<std::mutex> lk(g->mu);
    if (e != hipSuccess) {
        ws->busy = false;
        return from_hip(e);
    }
    ws->bytes = bytes;
    ws->cap = cap;
    return BC_OK;
}

void source_release(bc_graph_s *g, SourceWS *ws) {
    std::lock_guard<std::mutex> lk(g->mu);
    ws->busy = false;
}

// Pinned memory for a launch's tables; the kernels read them over the host
// link (a few words per workgroup), which costs less than a copy ahead of
// each launch.
bc_status source_tables(SourceWS *ws, size_t bytes) {
    if (ws->tab_cap >= bytes) return BC_OK;
    if (ws->h_tab) (void)hipHostFree(ws->h_tab);
    ws->h_tab = nullptr;
    ws->tab_cap = 0;
    BC_TRY_HIP(hipHostMalloc((void **)&ws->h_tab, bytes, hipHostMallocDefault));
    ws->tab_cap = bytes;
    return BC_OK;
}

SourceGraph source_graph(const bc_graph_s *g) {
    SourceGraph v{};
    v.n = g->n;
    v.cls[0] = 0;
    v.cls[1] = g->multi_end;
    v.cls[2] = g->big_end;
    v.cls[3] = g->mid_end;
    v.cls[4] = g->n;
    v.row_ptr = g->d_row_ptr;
    v.col_idx = g->d_col_idx;
    v.row_ptr_in = g->d_row_ptr_in;
    v.col_idx_in = g->d_col_idx_in;
    v.perm = g->d_perm;
    v.iperm = g->d_iperm;
    return v;
}

// Runs every job's requests: their units in as few launches as their scratch
// allows (one each for the undirected and the directed graphs of a round, with
// the values in LDS and in memory), then the rows of each request added in unit
// order.  Returns with all work finished; over[i] is set for a
// job with a count past double's range (its outputs then mean nothing).
bc_status source_jobs(const std::vector<SourceJob> &jobs, hipStream_t stream,
                      std::vector<char> &over) {
    const size_t nj = jobs.size();
    over.assign(nj, 0);
    struct Held {  // the jobs' workspaces, given back on every way out
        const std::vector<SourceJob> &jobs;
        std::vector<SourceWS *> ws;
        ~Held() {
            for (size_t j = 0; j < ws.size(); ++j)
                if (ws[j]) source_release(jobs[j].g, ws[j]);
        }
    } held{jobs, {}};
    // a unit: sources [first, first + count) of request `req`
    struct Unit {
        int32_t req, first, count;
    };
    std::vector<std::vector<Unit>> units(nj);
    std::vector<size_t> done(nj, 0), done_req(nj, 0);  // units and requests run
    size_t src_total = 0, req_total = 0, unit_room = 0;
    for (size_t j = 0; j < nj; ++j) {
        const SourceJob &job = jobs[j];
        for (size_t r = 0; r < job.reqs.size(); ++r) {
            const int32_t per = source_unit(job.g, job.reqs[r].k);
            for (int32_t a = 0; a < job.reqs[r].k; a += per)
                units[j].push_back({(int32_t)r, job.reqs[r].first + a,
                                    std::min(per, job.reqs[r].k - a)});
        }
        const int32_t cap = source_cap(job.g, (int64_t)units[j].size());
        held.ws.push_back(nullptr);
        const bc_status st = source_acquire(job.g, cap, &held.ws.back());
        if (st != BC_OK) {
            held.ws.pop_back();
            return st;
        }
        src_total += job.s_int.size();
        req_total += job.reqs.size();
        unit_room += std::min<size_t>(units[j].size(), (size_t)held.ws[j]->cap);
    }
    if (nj == 0) return BC_OK;
    SourceWS *tab = held.ws[0];
    size_t bytes = 0;
    auto part = [&](size_t b) {
        const size_t at = bytes;
        bytes += align_up(b);
        return at;
    };
    const size_t at_graphs = part(nj * sizeof(SourceGraph));
    const size_t at_units = part(std::max<size_t>(unit_room, 1) * sizeof(SourceUnit));
    const size_t at_sums = part(std::max<size_t>(req_total, 1) * sizeof(SourceSum));
    const size_t at_src = part(std::max<size_t>(src_total, 1) * sizeof(int32_t));
    const size_t at_rows = part(std::max<size_t>(src_total, 1) * sizeof(int32_t));
    const size_t at_range = part(nj * sizeof(int32_t));
    bc_status st = source_tables(tab, bytes);
    if (st != BC_OK) return st;
    SourceGraph *h_graphs = (SourceGraph *)(tab->h_tab + at_graphs);
    SourceUnit *h_units = (SourceUnit *)(tab->h_tab + at_units);
    SourceSum *h_sums = (SourceSum *)(tab->h_tab + at_sums);
    int32_t *h_src = (int32_t *)(tab->h_tab + at_src);
    int32_t *h_rows = (int32_t *)(tab->h_tab + at_rows);
    int32_t *h_range = (int32_t *)(tab->h_tab + at_range);
    std::vector<int32_t> src_at(nj);
    {
        int32_t at = 0;
        for (size_t j = 0; j < nj; ++j) {
            h_graphs[j] = source_graph(jobs[j].g);
            h_range[j] = 0;
            src_at[j] = at;
            std::copy(jobs[j].s_int.begin(), jobs[j].s_int.end(), h_src + at);
            if (jobs[j].export_row)
                std::copy(jobs[j].export_row, jobs[j].export_row + jobs[j].s_int.size(), h_rows + at);
            at += (int32_t)jobs[j].s_int.size();
        }
    }
    // measurement: single-graph calls only
    bc_graph_s *pg = nj == 1 ? jobs[0].g : nullptr;
    const bool prof = pg && pg->profiling.load() != 0;
    LaunchTimer timer;
    timer.on = prof;
    unsigned long long *d_stats = nullptr;
    if (prof) {
        if (!tab->d_stats) BC_TRY_HIP(hipMalloc(&tab->d_stats, kStatWords * sizeof(unsigned long long)));
        d_stats = tab->d_stats;
        BC_TRY_HIP(hipMemsetAsync(d_stats, 0, kStatWords * sizeof(unsigned long long), stream));
    }
    hipError_t e = hipSuccess;
    bool more = true;
    while (more && e == hipSuccess) {
        more = false;
        // the round's units, the undirected graphs' first, and the sums of the
        // requests they belong to
        size_t nu = 0, ns = 0;
        int32_t max_n = 0;
        struct Launch {
            size_t first, count;
            size_t lds;
        } launch[4];
        std::vector<size_t> take(nj, 0);
        for (size_t j = 0; j < nj; ++j) {
            const SourceJob &job = jobs[j];
            const size_t per = source_unit_bytes(job.g);
            // whole requests while they fit; one sum per request (of no rows
            // for one without sources: its BC is zero), except that a lone
            // unit writes its request's BC itself
            for (; done_req[j] < job.reqs.size(); ++done_req[j]) {
                const SourceReq &rq = job.reqs[done_req[j]];
                size_t k = 0;
                while (done[j] + take[j] + k < units[j].size() &&
                       units[j][done[j] + take[j] + k].req == (int32_t)done_req[j])
                    ++k;
                if (take[j] + k > (size_t)held.ws[j]->cap) break;
                const size_t at = take[j];
                take[j] += k;
                if (k == 1) continue;
                SourceSum &s = h_sums[ns++];
                s.n = job.g->n;
                s.units = (int32_t)k;
                s.stride = per / sizeof(double);
                s.row = (const double *)((char *)held.ws[j]->block + at * per);
                s.iperm = job.g->d_iperm;
                s.out = rq.out;
                max_n = std::max(max_n, job.g->n);
            }
            more |= done_req[j] < job.reqs.size();
        }
        for (int kind = 0; kind < 4; ++kind) {
            Launch &l = launch[kind];
            l = {nu, 0, 0};
            for (size_t j = 0; j < nj; ++j) {
                const SourceJob &job = jobs[j];
                if (kind != (job.g->directed ? 1 : 0) + (source_in_lds(job.g->n) ? 0 : 2)) continue;
                if (take[j] == 0) continue;
                const size_t n = (size_t)job.g->n;
                const size_t per = source_unit_bytes(job.g);
                l.lds = std::max(l.lds, source_lds_bytes(job.g->n));
                for (size_t i = 0; i < take[j]; ++i) {
                    const Unit &un = units[j][done[j] + i];
                    const SourceReq &rq = job.reqs[(size_t)un.req];
                    SourceUnit &d = h_units[nu++];
                    char *p = (char *)held.ws[j]->block + i * per;
                    auto cut = [&](size_t b) {
                        char *q = p;
                        p += align_up(b);
                        return (void *)q;
                    };
                    d.graph = (int32_t)j;
                    d.first = src_at[j] + un.first;
                    d.count = un.count;
                    d.row = (double *)cut(n * sizeof(double));
                    d.q = (int32_t *)cut(n * sizeof(int32_t));
                    d.lvl = (uint32_t *)cut((n + 2) * kSrcClasses * sizeof(uint32_t));
                    d.sig = (double *)cut(n * sizeof(double));  // (the last of them)
                    d.out = un.count == rq.k ? rq.out : nullptr;
                    d.dist = job.dist;
                    d.sigma = job.sigma;
                    d.export_row = h_rows + d.first;
                }
                done[j] += take[j];
            }
            l.count = nu - l.first;
        }
        for (int kind = 0; kind < 4 && e == hipSuccess; ++kind) {
            const Launch &l = launch[kind];
            if (l.count == 0) continue;
            e = timer.begin(BC_PROF_FUSED, stream);
            if (e == hipSuccess)
                e = source_run(h_units + l.first, (int32_t)l.count, h_graphs, h_src, kind % 2 == 1,
                               kind < 2, l.lds, h_range, d_stats, stream);
            if (e == hipSuccess) e = timer.end(stream);
        }
        if (e == hipSuccess) e = source_sum(h_sums, (int32_t)ns, max_n, stream);
        // (the tables are rewritten by the next round)
        const hipError_t es = hipStreamSynchronize(stream);
        if (e == hipSuccess) e = es;
    }
    if (e == hipSuccess) {
        for (size_t j = 0; j < nj; ++j) over[j] = h_range[j] != 0;
        if (prof) {
            unsigned long long depths = 0;
            e = hipMemcpy(&depths, d_stats + 14, sizeof depths, hipMemcpyDeviceToHost);
            accumulate_profile(pg, timer, d_stats, 2 * (int64_t)depths + (int64_t)src_total);
        }
    }
    timer.destroy();
    return from_hip(e);
}

// Estimated times of a call's alternatives in seconds, fitted to measured
// calls (MI355X, R-MAT of 4K to 131K vertices with edge factors 4 to 100,
// uniform random of 1K to 100K with 4 to 900 arcs per vertex, directed R-MAT;
// 1 to 16,384 sources).  For instance, ms on the host loop and here,
//   values in LDS, 64 sources: uniform random of 20K vertices with 50 arcs each
//     0.37 / 0.50, with 16 0.75 / 0.35; R-MAT of 16K vertices with edge factor
//     64 0.62 / 0.62, with 16 0.68 / 0.28
//   values in memory, 64 and 4,096 sources: uniform random of 21K vertices with
//     4 arcs each 1.24 / 0.26 and 40 / 6.3; 50K with 4 1.34 / 0.64 and 43 / 22,
//     with 16 1.06 / 1.85 and 39 / 76; 100K with 4 1.37 / 1.36 and 49 / 54;
//     R-MAT of 33K vertices, edge factor 4 0.75 / 0.36 and 20.6 / 6.8, 65K
//     0.85 / 0.75 and 22.0 / 17.9, 131K 0.94 / 1.80 and 27 / 48
//
// A graph whose arcs gather at few vertices, against one of even degrees.
static bool skewed(const bc_graph_s *g) {
    return g->arc_degree * (double)std::max(g->live_end, 1) > 2.0 * (double)g->nnz;
}

// This path: rounds of as many sources as the device holds, by vertices and arcs
// (more where two workgroups share a compute unit, where a directed graph's
// forward pass reads two rows, and where rows end just past a turn of 64 arcs;
// less where the ids are those of few vertices).  With the values in memory a
// time per source, and more as a round's 256 sources fill the L2s, a fifth of
// that where hubs keep to few lines; with a margin, as its estimate varies more.
static double source_seconds(const bc_graph_s *g, int32_t k) {
    const double n = (double)g->n, arcs = (double)g->nnz;
    const double degree = arcs / (double)std::max(g->live_end, 1);
    if (!source_in_lds(g->n)) {
        const double crowd = (skewed(g) ? 0.44e-9 : 2.2e-9) * (g->directed ? 1.7 : 1.0) *
                             std::pow(n / 21000.0, 0.67) * arcs;
        const double round = 4e-9 * n + 1.0e-9 * arcs + crowd * std::min(1.0, (double)k / kCus);
        return (50e-6 + std::max(1.0, (double)k / kCus) * round) / 0.85;
    }
    const int32_t per = source_per_cu(g);
    const double rounds = std::ceil((double)k / ((double)kCus * per));
    double arc = (g->directed ? 0.45e-9 : 0.35e-9) * std::min(1.0, n / 8192.0);
    if (!skewed(g) && degree > 64.0) arc *= std::ceil(degree / 64.0) * 64.0 / degree;
    return 25e-6 + rounds * (25e-6 + (6e-9 * n + arc * arcs) * (k > kCus && per > 1 ? 1.4 : 1.0));
}

// Host loop: a time per level of a batch, more where degrees are even and small,
// the levels by degree (the breadth of a uniform random graph, with a tail and
// six more where degrees are skewed).  A batch of fewer sources takes less where levels are thin;
// batches run four at once, sparse ones beside each other more easily.
static double host_seconds(const bc_graph_s *g, int32_t k) {
    const double arcs = (double)g->nnz, live = std::max(g->live_end, 2);
    const double degree = std::max(arcs / live, 1.5);
    const double breadth = 1.3 + std::log(live) / std::log(degree);
    const bool skew = skewed(g), thin = !skew && degree < 32.0;
    const double few = std::min(1.0, 256.0 / (degree * degree));
    const double levels = skew ? 0.045e-3 * (breadth + 2.0 * std::log(live) / degree + 6.0)
                               : (0.05e-3 + 0.078e-3 * few) * breadth;
    const double batch = levels + 0.115e-9 * arcs + 3e-9 * (double)g->n;
    const double batches = std::ceil((double)k / kWave);
    if (batches <= 1.0) return batch * std::pow((double)k / kWave, thin ? 0.25 : 0.1);
    return batch * (skew ? 0.5 + 0.4 * batches : (thin ? 0.5 + 0.5 * batches : 0.4 + 0.65 * batches));
}

// Few sources, where the one-source path is the alternative (R-MAT of 1K to
// 16K vertices: 0.154, 0.166 and 0.185 ms for one, 0.10 .. 0.14 ms for each of
// many; here 0.475 ms for one alone at 426K arcs, which waits for its arcs to
// reach its L2, and 0.28 for several).  Beyond 1.3M arcs that path is faster
// than this estimate of it (uniform random of 20K vertices with 100 arcs each,
// 8 sources: 0.75 ms against 1.04).
bool source_beats_plain(const bc_graph_s *g, int32_t k) {
    const double arcs = (double)g->nnz;
    const double here = source_in_lds(g->n) ? 50e-6 + (k == 1 ? 1.0e-9 : 0.6e-9) * arcs
                                            : source_seconds(g, k);
    return arcs < 1.3e6 && here < 50e-6 + (double)k * (0.105e-3 + 40e-12 * arcs);
}

// Whether a batched call of k sources takes this path.  `shared`: the call's
// other graphs run beside these sources here, but one after the other on the
// host loop.
bool use_source(const bc_graph_s *g, int32_t level_loop, int32_t k, int32_t width, bool shared) {
    if (g->sigma_ext.load()) return false;  // extended range: host loop only
    if (width > kWave) return false;        // two lane words per vertex: host loop only
    if (!source_fits(g)) return false;
    if (level_loop == BC_LOOP_HOST || level_loop == BC_LOOP_GRAPH) return false;
    const bool lds = source_in_lds(g->n);
    if (level_loop == BC_LOOP_DEVICE && lds) return true;
    if (level_loop == BC_LOOP_AUTO && !shared && !lds && g->deep) return false;  // as queues
    // (a graph that joins others in a call runs here alone under DEVICE, too)
    const bool lean = shared || level_loop == BC_LOOP_DEVICE;
    if (source_seconds(g, k) < (lean ? (lds ? 1.8 : 1.3) : 1.0) * host_seconds(g, k)) return true;
    // (for few sources the other choice is one at a time, not the host loop)
    return !g->directed && k < g->tuned_min_batched.load() && source_beats_plain(g, k);
}

// By the 64-source call, and with the values in memory by the one-source call
// too, which loses more there than it would with them in LDS.
bool multi_source(const bc_graph_s *g) {
    if (source_in_lds(g->n)) return use_source(g, BC_LOOP_AUTO, kWave, kWave, true);
    return use_source(g, BC_LOOP_DEVICE, kWave, kWave) &&
           source_seconds(g, kWave) < host_seconds(g, kWave) &&
           source_seconds(g, 1) < 1.3 * host_seconds(g, 1);
}

// (a unit per source: what a call of many small requests takes)
size_t source_bytes(const bc_graph_s *g, int32_t k) {
    return (size_t)source_cap(g, k) * source_unit_bytes(g);
}

}  // namespace bcx
