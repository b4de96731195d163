// Host side of the batched path: batch workspaces, batch composition
// (landmark order), the host-driven level loop, concurrent parts and
// multi-request batching.
#include "bc_runtime.h"

namespace bcx {

// Chunk items with a partial row: both passes' items (the forward pass runs
// over the arcs into each vertex, the reverse pass over the arcs out of it).
size_t partial_rows(const bc_graph_s::BcItems &t) {
    return (size_t)std::max<uint32_t>(std::max(t.items, t.items_in), 1);
}

size_t partial_rows(const bc_graph_s *g) { return partial_rows(g->bci); }

// The batched path's work items of a workspace: tables t.
void set_items(const bc_graph_s::BcItems &t, BatchDev &d) {
    d.big_end = t.big_end;
    d.multi_end = t.multi_end;
    d.chunk = t.chunk;
    d.items = t.items;
    d.item_info = t.info;
    d.item_first = t.first;
    d.items_in = t.items_in;
    d.item_info_in = t.info_in;
    d.item_first_in = t.first_in;
}

// ... the graph's current tables (the host-driven loop's).
void set_items(const bc_graph_s *g, BatchDev &d) { set_items(g->bci, d); }

// Rows of the graph's counts: double once a count passed 32 bits (or the
// extended range is on), uint32 before.
bool sigma_rows_wide(const bc_graph_s *g) { return g->sigma_wide.load() || g->sigma_ext.load(); }

size_t batch_ws_bytes_rows(const bc_graph_s *g, int32_t H, bool wide) {
    const size_t n = (size_t)std::max<int32_t>(g->n, 1);
    const size_t lanes = (size_t)H * kWave;
    size_t b = 0;
    b += align_up(n * H * sizeof(uint64_t));             // vis
    b += align_up(n * lanes * (wide ? sizeof(double) : sizeof(uint32_t)));  // sigma rows
    b += align_up(n * lanes * sizeof(double));           // coef rows
    b += align_up(kBatchCtrlInts * sizeof(int32_t));     // ctrl
    b += align_up(n * H * sizeof(double));               // bc, one array per half
    b += align_up((size_t)std::max(g->bci.multi_end, 1) * H * sizeof(uint64_t));  // reach
    b += align_up(partial_rows(g) * lanes * sizeof(double));  // chunk partial rows
    b += align_up(kStatWords * sizeof(unsigned long long));     // work counters
    b += align_up(n * sizeof(int32_t));                  // candidate list
    // item list of the sparse step (the forward pass's items)
    b += align_up((size_t)std::max<uint32_t>(g->bci.items_in, 1) * sizeof(int32_t));
    b += align_up((size_t)kFrontSets * kFrontWaves * 2 * sizeof(unsigned long long));
    b += align_up(((n + 15) / 16) * 16);                 // candidate marks
    return b;
}

size_t batch_ws_bytes(const bc_graph_s *g, int32_t H) {
    return batch_ws_bytes_rows(g, H, sigma_rows_wide(g));
}

// F[lcap][n][H] and the extended-range tables xs, xmax, xe ([lcap][H][64] each).
size_t batch_level_bytes(const bc_graph_s *g, int32_t lcap, int32_t H) {
    return (size_t)lcap * H *
           ((size_t)std::max<int32_t>(g->n, 1) * sizeof(uint64_t) +
            kWave * (sizeof(double) + sizeof(unsigned long long) + sizeof(int32_t)));
}

void batch_ws_destroy(BatchWS *ws) {
    if (!ws) return;
    if (ws->done) {
        (void)hipEventSynchronize(ws->done);
        (void)hipEventDestroy(ws->done);
    }
    ws->timer.destroy();
    if (ws->F) (void)hipFree(ws->F);
    if (ws->d_src) (void)hipFree(ws->d_src);
    if (ws->wide_sigma) (void)hipFree(ws->wide_sigma);
    if (ws->block) (void)hipFree(ws->block);
    if (ws->h_ctrl) (void)hipHostFree(ws->h_ctrl);
    delete ws;
}

bc_status batch_ws_create(bc_graph_s *g, int32_t H, BatchWS **out) {
    BatchWS *ws = new (std::nothrow) BatchWS();
    if (!ws) return BC_ERR_OUT_OF_MEMORY;
    ws->H = H;
    ws->gen = g->bci_gen.load();
    ws->wide = sigma_rows_wide(g);  // read once: the layout below follows it
    ws->bytes = batch_ws_bytes_rows(g, H, ws->wide);
    hipError_t e = hipMalloc(&ws->block, ws->bytes);
    if (e == hipSuccess)
        e = hipHostMalloc((void **)&ws->h_ctrl, kBatchCtrlInts * sizeof(int32_t),
                          hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ws->done, hipEventDisableTiming);
    if (e != hipSuccess) {
        batch_ws_destroy(ws);
        return from_hip(e);
    }
    const size_t n = (size_t)std::max<int32_t>(g->n, 1);
    char *p = (char *)ws->block;
    auto take = [&](size_t bytes) {
        char *r = p;
        p += align_up(bytes);
        return (void *)r;
    };
    BatchDev &d = ws->dev;
    const size_t lanes = (size_t)H * kWave;
    d.n = g->n;
    d.H = H;
    d.row_ptr = g->d_row_ptr;
    d.col_idx = g->d_col_idx;
    d.vis = (uint64_t *)take(n * H * sizeof(uint64_t));
    d.sigma = (double *)take(n * lanes * (ws->wide ? sizeof(double) : sizeof(uint32_t)));
    d.sigma32 = reinterpret_cast<uint32_t *>(d.sigma);
    d.narrow = 1;
    d.coef = (double *)take(n * lanes * sizeof(double));
    d.ctrl = (int32_t *)take(kBatchCtrlInts * sizeof(int32_t));
    d.bc = (double *)take(n * H * sizeof(double));
    d.reach = (uint64_t *)take((size_t)std::max(g->bci.multi_end, 1) * H * sizeof(uint64_t));
    d.partial = (double *)take(partial_rows(g) * lanes * sizeof(double));
    set_items(g, d);
    d.row_ptr_in = g->d_row_ptr_in;
    d.col_idx_in = g->d_col_idx_in;
    ws->d_stats = (unsigned long long *)take(kStatWords * sizeof(unsigned long long));
    d.stats = nullptr;
    d.clist = (int32_t *)take(n * sizeof(int32_t));
    d.ilist = (int32_t *)take((size_t)std::max<uint32_t>(g->bci.items_in, 1) * sizeof(int32_t));
    d.cand = (uint8_t *)take(((n + 15) / 16) * 16);
    d.front = (unsigned long long *)take((size_t)kFrontSets * kFrontWaves * 2 *
                                         sizeof(unsigned long long));
    d.nnz = g->nnz;
    d.sparse_arcs = g->nnz / kDefaultSparseDiv;
    d.F = nullptr;
    d.lcap = 0;
    *out = ws;
    return BC_OK;
}

// Double-sized sigma rows for a workspace built with uint32 ones (its own
// region stays unused).
bc_status batch_widen(bc_graph_s *g, BatchWS *ws) {
    if (ws->wide) return BC_OK;
    const size_t bytes = (size_t)std::max<int32_t>(g->n, 1) * ws->H * kWave * sizeof(double);
    BC_TRY_HIP(hipMalloc(&ws->wide_sigma, bytes));
    ws->wide = true;
    ws->bytes += bytes;
    ws->dev.sigma = (double *)ws->wide_sigma;
    ws->dev.sigma32 = reinterpret_cast<uint32_t *>(ws->wide_sigma);
    return BC_OK;
}

bc_status batch_grow_levels(bc_graph_s *g, BatchWS *ws, int32_t lcap) {
    if (lcap <= ws->lcap) return BC_OK;
    if (ws->F) (void)hipFree(ws->F);
    ws->F = nullptr;
    ws->lcap = 0;
    const int32_t H = ws->H;
    BC_TRY_HIP(hipMalloc(&ws->F, batch_level_bytes(g, lcap, H)));
    ws->lcap = lcap;
    ws->dev.F = ws->F;
    ws->dev.lcap = lcap;
    ws->xs = (double *)(ws->F + (size_t)lcap * H * (size_t)std::max<int32_t>(g->n, 1));
    ws->xmax = (unsigned long long *)(ws->xs + (size_t)lcap * H * kWave);
    ws->xe = (int32_t *)(ws->xmax + (size_t)lcap * H * kWave);
    return BC_OK;
}

bc_status batch_acquire(bc_graph_s *g, int32_t H, hipStream_t stream, BatchWS **out) {
    {
        std::lock_guard<std::mutex> lk(g->mu);
        for (BatchWS *ws : g->batch_pool) {
            if (!ws->busy && ws->H == H && ws->gen == g->bci_gen.load()) {
                ws->busy = true;
                *out = ws;
                BC_TRY_HIP(hipStreamWaitEvent(stream, ws->done, 0));
                return BC_OK;
            }
        }
    }
    BatchWS *ws = nullptr;
    bc_status st = batch_ws_create(g, H, &ws);
    if (st != BC_OK) return st;
    ws->busy = true;
    std::lock_guard<std::mutex> lk(g->mu);
    g->batch_pool.push_back(ws);
    *out = ws;
    return BC_OK;
}

void batch_release(bc_graph_s *g, BatchWS *ws, hipStream_t stream) {
    (void)hipEventRecord(ws->done, stream);
    std::lock_guard<std::mutex> lk(g->mu);
    ws->busy = false;
}

bc_status ensure_landmarks(bc_graph_s *g) {
    std::lock_guard<std::mutex> lk(g->land_mu);
    if (g->land_ready) return BC_OK;
    if (g->n == 0) {
        g->land_ready = true;
        return BC_OK;
    }
    bc_status st = bfs_levels(g, 0, g->land1);
    if (st != BC_OK) return st;
    int32_t far = 0;
    for (int32_t v = 0; v < g->n; ++v)
        if (g->land1[(size_t)v] > g->land1[(size_t)far]) far = v;
    st = bfs_levels(g, far, g->land2);
    if (st != BC_OK) return st;
    g->land_ready = true;
    return BC_OK;
}

constexpr size_t kMaxChunkGraphs = 16;

ChunkGraphs::~ChunkGraphs() {
    for (Entry &e : entries)
        if (e.exec) (void)hipGraphExecDestroy(e.exec);
    if (cap) (void)hipStreamDestroy(cap);
}

hipError_t ChunkGraphs::replay(const BatchDev &d, int32_t dir, int32_t K, int32_t nlanes,
                               hipStream_t stream) {
    Entry *hit = nullptr;
    for (Entry &en : entries)
        if (en.dir == dir && en.K == K && en.nlanes == nlanes &&
            std::memcmp(&en.d, &d, sizeof(BatchDev)) == 0) {
            hit = &en;
            break;
        }
    if (!hit) {
        if (!cap) {
            const hipError_t ec = hipStreamCreateWithFlags(&cap, hipStreamNonBlocking);
            if (ec != hipSuccess) return ec;
        }
        // kernel launches only (no memset nodes): K relative steps, then the
        // base moved by K levels
        hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return e;
        for (int32_t i = 0; i < K && e == hipSuccess; ++i) {
            const int32_t L = kRelLevel + i;
            if (dir > 0) {
                e = batch_forward(d, L, nlanes, cap);
                if (e == hipSuccess) e = batch_forward_done(d, L, cap);
            } else {
                e = batch_reverse(d, L, cap);
                if (e == hipSuccess) e = batch_finalize_rel(d, L, cap);
            }
        }
        if (e == hipSuccess) e = batch_level_advance(d, dir * K, cap);
        hipGraph_t graph = nullptr;
        const hipError_t ee = hipStreamEndCapture(cap, &graph);
        if (e == hipSuccess) e = ee;
        hipGraphExec_t exec = nullptr;
        if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (graph) (void)hipGraphDestroy(graph);
        if (e != hipSuccess) return e;
        if (entries.size() >= kMaxChunkGraphs) {
            // every earlier launch of the workspace's graphs is ordered before
            // this stream's current work (the workspace is acquired on it)
            e = hipStreamSynchronize(stream);
            if (e != hipSuccess) {
                (void)hipGraphExecDestroy(exec);
                return e;
            }
            (void)hipGraphExecDestroy(entries.front().exec);
            entries.erase(entries.begin());
        }
        Entry en;
        en.dir = dir;
        en.K = K;
        en.nlanes = nlanes;
        en.d = d;
        en.exec = exec;
        entries.push_back(en);
        hit = &entries.back();
    }
    return hipGraphLaunch(hit->exec, stream);
}

// One batch: clear and seed, the forward levels in chunks with one host poll
// per chunk, then the reverse levels.  A path count that needs double rows
// (or the extended range) switches the graph to them and asks for a rerun; a
// level array too short for the batch asks for a longer one.  With cg, each
// chunk of levels is one replayed graph instead of its launches.
hipError_t drive_batch(bc_graph_s *g, BatchDev &d, const ExtTables &ext, const int32_t *lanes_dev,
                       int32_t nl, int32_t *h_ctrl, hipStream_t stream, LaunchTimer &timer,
                       unsigned long long *d_stats, int32_t stride, BatchOutcome &how,
                       int32_t &deepest, ChunkGraphs *cg, bool wide_ok) {
    const int32_t n = g->n;
    const bool prof = d_stats != nullptr;
    auto measure = [&](int32_t L) {
        const bool m = prof && L % stride == 0;
        timer.on = m;
        d.stats = m ? d_stats : nullptr;
    };
    const bool use_ext = g->sigma_ext.load();
    const bool wide = use_ext || g->sigma_wide.load();
    how = BatchOutcome::Done;
    deepest = 0;
    if (wide && !wide_ok) {  // uint32-sized rows cannot take double counts
        how = BatchOutcome::NeedWide;
        return hipSuccess;
    }
    d.narrow = wide ? 0 : 1;
    d.xs = use_ext ? ext.xs : nullptr;
    d.xmax = use_ext ? ext.xmax : nullptr;
    d.xe = use_ext ? ext.xe : nullptr;
    hipError_t e = batch_start(d, lanes_dev, nl, stream);
    if (e != hipSuccess) return e;
    int32_t L0 = 0;
    for (;;) {
        const int32_t K = std::max(2, g->batch_depth_hint.load() + 2);
        const int32_t Lend = std::min(L0 + K, d.lcap - 1);
        // (a replayed chunk runs levels L0 .. L0+K-1; those past the level
        // array's end return at once, as the host loop would not launch them)
        if (cg) e = cg->replay(d, 1, K, nl, stream);
        for (int32_t L = L0; !cg && L < Lend && e == hipSuccess; ++L) {
            measure(L);
            e = timer.begin(BC_PROF_FORWARD, stream);
            if (e == hipSuccess) e = batch_forward(d, L, nl, stream);
            if (e == hipSuccess) e = timer.end(stream);
            if (e == hipSuccess) e = timer.begin(BC_PROF_COMPACT, stream);
            if (e == hipSuccess) e = batch_forward_done(d, L, stream);
            if (e == hipSuccess) e = timer.end(stream);
        }
        if (e == hipSuccess)
            e = hipMemcpyAsync(h_ctrl, d.ctrl, kBatchCtrlInts * sizeof(int32_t),
                               hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return e;
        deepest = h_ctrl[kCtlDeepest];
        if (h_ctrl[kCtlNarrow]) {  // a path count needs double rows: run again
            g->sigma_wide.store(true);
            how = BatchOutcome::Rerun;
            return hipSuccess;
        }
        if (h_ctrl[kCtlRange] && !use_ext) {  // beyond double: run again level-scaled
            g->sigma_wide.store(true);
            g->sigma_ext.store(true);
            how = BatchOutcome::Rerun;
            return hipMemsetAsync(d.ctrl + kCtlRange, 0, sizeof(int32_t), stream);
        }
        if (h_ctrl[kCtlTrunc]) {
            how = BatchOutcome::Grow;
            return hipSuccess;
        }
        if (deepest < Lend || Lend >= n) break;
        L0 = Lend;
    }
    if (cg) {
        // chunks of K levels from the deepest one down (levels below 1 return
        // at once); the first chunk's base is the deepest level
        const int32_t K = std::max(2, g->batch_depth_hint.load() + 2);
        if (deepest >= 1) e = batch_level_from_deepest(d, stream);
        for (int32_t done = 0; done < deepest && e == hipSuccess; done += K)
            e = cg->replay(d, -1, K, 0, stream);
        return e;
    }
    for (int32_t L = deepest; L >= 1 && e == hipSuccess; --L) {
        measure(L);
        if (L != deepest) {
            e = timer.begin(BC_PROF_REVERSE, stream);
            if (e == hipSuccess) e = batch_reverse(d, L, stream);
            if (e == hipSuccess) e = timer.end(stream);
        }
        if (e == hipSuccess) e = timer.begin(BC_PROF_FINISH, stream);
        if (e == hipSuccess) e = batch_finalize(d, L, L == deepest, stream);
        if (e == hipSuccess) e = timer.end(stream);
    }
    return e;
}

// One batch of a batched run: lanes [first, first + nlanes) of the run's
// (internal-id) source list; with nseg > 0, its lanes feed nseg request
// outputs described from seg_first on in the run's segment tables.
struct BatchPlan {
    int32_t first, nlanes;
    int32_t seg_first, nseg;
};

// Execute a batch plan.  s_int: internal source ids in lane order.  With
// nseg == 0 everywhere, BC accumulates in the workspace and is gathered into
// bc_out (caller order); otherwise each segment's output (caller order,
// zeroed by the caller) receives its lanes' dependencies.  export_row maps a
// lane of the run to the dist / sigma export row (or NULL: no export).
bc_status run_batch_plan(bc_graph_s *g, const std::vector<int32_t> &s_int,
                         const std::vector<BatchPlan> &plan,
                         const std::vector<int32_t> &seg_start,  // per segment table: nseg+1
                         const std::vector<double *> &seg_out, double *bc_out,
                         hipStream_t stream, const int32_t *export_row, int32_t *dist,
                         double *sigma, int32_t sparse_div, bool graphs) {
    // two lane words per vertex when a batch has more than 64 sources (never
    // with request segments: their lanes are summed within one 64-lane word)
    int32_t H = 1;
    for (const BatchPlan &bp : plan) H = std::max(H, bp.nlanes > kWave ? 2 : 1);
    BatchWS *ws = nullptr;
    bc_status st = batch_acquire(g, H, stream, &ws);
    if (st != BC_OK) return st;
    auto fail = [&](bc_status s2) {
        batch_release(g, ws, stream);
        return s2;
    };
    const int32_t n = g->n;
    const int32_t k = (int32_t)s_int.size();
    const bool prof = g->profiling.load() != 0;
    ws->dev.stats = prof ? ws->d_stats : nullptr;
    ws->timer.on = prof;
    ws->timer.used = 0;
    // frontier arcs below which a level takes the sparse step (0: never); the
    // halves of a two-word batch count their frontiers separately
    ws->dev.sparse_arcs = sparse_div < 0 ? 0 : H * (g->nnz / std::max(sparse_div, 1));
    if (prof) {
        hipError_t ez = hipMemsetAsync(ws->d_stats, 0, kStatWords * sizeof(unsigned long long), stream);
        if (ez != hipSuccess) return fail(from_hip(ez));
    }
    st = batch_grow_levels(g, ws, std::max(ws->lcap, g->batch_depth_hint.load() + 8));
    if (st != BC_OK) return fail(st);
    // device copies of the lane sources and the segment tables
    const size_t seg_ints = seg_start.size(), seg_ptrs = seg_out.size();
    const size_t need = (size_t)k * sizeof(int32_t) + seg_ints * sizeof(int32_t) +
                        seg_ptrs * sizeof(double *) + 64;
    if (need > ws->src_cap) {
        if (ws->d_src) (void)hipFree(ws->d_src);
        ws->d_src = nullptr;
        ws->src_cap = 0;
        hipError_t ea = hipMalloc(&ws->d_src, need);
        if (ea != hipSuccess) return fail(from_hip(ea));
        ws->src_cap = need;
    }
    int32_t *d_lanes = ws->d_src;
    int32_t *d_seg_start = d_lanes + k;
    double **d_seg_out =
        (double **)(((uintptr_t)(d_seg_start + seg_ints) + 15) & ~(uintptr_t)15);
    int32_t *x_dist = nullptr;
    double *x_sigma = nullptr;
    struct Tmp {
        int32_t *&a;
        double *&b;
        ~Tmp() {
            if (a) (void)hipFree(a);
            if (b) (void)hipFree(b);
        }
    } tmp_guard{x_dist, x_sigma};
    hipError_t e = hipSuccess;
    if (dist) e = hipMalloc(&x_dist, (size_t)H * kWave * (size_t)n * sizeof(int32_t));
    if (e == hipSuccess && sigma)
        e = hipMalloc(&x_sigma, (size_t)H * kWave * (size_t)n * sizeof(double));
    if (e == hipSuccess && k > 0)
        e = hipMemcpyAsync(d_lanes, s_int.data(), (size_t)k * sizeof(int32_t),
                           hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && seg_ints)
        e = hipMemcpyAsync(d_seg_start, seg_start.data(), seg_ints * sizeof(int32_t),
                           hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && seg_ptrs)
        e = hipMemcpyAsync(d_seg_out, seg_out.data(), seg_ptrs * sizeof(double *),
                           hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && bc_out)
        e = hipMemsetAsync(ws->dev.bc, 0, (size_t)H * n * sizeof(double), stream);
    if (e == hipSuccess)  // the batches' kernels only ever set the range flag
        e = hipMemsetAsync(ws->dev.ctrl + kCtlRange, 0, sizeof(int32_t), stream);
    if (e != hipSuccess) return fail(from_hip(e));
    int32_t range = 0, run_depth = 0;
    int64_t level_steps = 0;  // forward and reverse, over the batches
    // measurement covers the launches of every stride-th level only (all of
    // them with stride 1): events around every launch slow deep graphs' short
    // level steps
    const int32_t stride = std::max(1, g->profiling.load());
    for (size_t bi = 0; bi < plan.size();) {
        const BatchPlan &bp = plan[bi];
        const int32_t nl = bp.nlanes;
        BatchDev &d = ws->dev;
        d.nseg = bp.nseg;
        d.seg_start = bp.nseg ? d_seg_start + bp.seg_first : nullptr;
        d.seg_out = bp.nseg ? d_seg_out + (bp.seg_first - (int32_t)bi) : nullptr;
        d.iperm = g->d_iperm;
        BatchOutcome how = BatchOutcome::Done;
        int32_t deepest = 0;
        const ExtTables ext{ws->xs, ws->xmax, ws->xe};
        // (measured runs launch every step: the events go around each launch)
        e = drive_batch(g, d, ext, d_lanes + bp.first, nl, ws->h_ctrl, stream, ws->timer,
                        prof ? ws->d_stats : nullptr, stride, how, deepest,
                        graphs && !prof ? &ws->graphs : nullptr, ws->wide);
        if (e != hipSuccess) return fail(from_hip(e));
        if (how == BatchOutcome::NeedWide) {  // double rows from now on
            st = batch_widen(g, ws);
            if (st != BC_OK) return fail(st);
            continue;
        }
        if (how == BatchOutcome::Rerun) continue;
        if (how == BatchOutcome::Grow) {  // level array full: grow it, run the batch again
            st = batch_grow_levels(g, ws, ws->lcap * 2);
            if (st != BC_OK) return fail(st);
            continue;
        }
        if (e == hipSuccess && export_row && (dist || sigma)) {
            e = batch_export(d, deepest, nl, x_dist, x_sigma, stream);
            for (int32_t s2 = 0; s2 < nl && e == hipSuccess; ++s2) {
                const size_t row = (size_t)export_row[bp.first + s2] * (size_t)n;
                if (dist) e = gather_i32(n, g->d_perm, x_dist + (size_t)s2 * n, dist + row, stream);
                if (e == hipSuccess && sigma)
                    e = gather_f64(n, g->d_perm, x_sigma + (size_t)s2 * n, sigma + row, stream);
            }
        }
        if (e != hipSuccess) return fail(from_hip(e));
        range |= ws->h_ctrl[1];
        run_depth = std::max(run_depth, deepest);
        level_steps += 2 * (int64_t)deepest + 1;
        ++bi;
    }
    ws->dev.nseg = 0;
    // the halves' BC arrays added (half 0 + half 1, in place)
    if (bc_out && H > 1) e = sum_parts(n, ws->dev.bc, H, ws->dev.bc, stream);
    if (e == hipSuccess && bc_out) e = gather_f64(n, g->d_perm, ws->dev.bc, bc_out, stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ws->h_ctrl, ws->dev.ctrl, kBatchCtrlInts * sizeof(int32_t),
                           hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fail(from_hip(e));
    range |= ws->h_ctrl[1];
    if (k > 0) g->batch_depth_hint.store(run_depth);
    if (prof) accumulate_profile(g, ws->timer, ws->d_stats, level_steps);
    batch_release(g, ws, stream);
    return range ? BC_ERR_RANGE : BC_OK;
}

// Several graphs in one call: the sources of the graphs that join go in one
// launch, a workgroup per source (one launch per kind of graph); every
// graph's BC is made of the same units as its own run's, so it is
// bit-identical to it.  A graph that cannot join (extended range, too large)
// or whose counts pass double's range runs on its own afterwards.
bc_status run_graphs(bc_graph_s *const *gs, int32_t ng, const int32_t *const *sources,
                     const int32_t *ks, double *const *outs, int32_t level_loop,
                     int32_t *loops, hipStream_t stream) {
    std::vector<char> join((size_t)ng, 0);
    for (int32_t i = 0; i < ng; ++i)
        join[(size_t)i] = use_source(gs[i], level_loop, ks[i], kWave, ng > 1);
    std::vector<SourceJob> jobs;
    std::vector<int32_t> at, alone;
    for (int32_t i = 0; i < ng; ++i) {
        bc_graph_s *g = gs[i];
        if (g->n == 0) continue;
        if (!join[(size_t)i]) {
            alone.push_back(i);
            continue;
        }
        SourceJob job;
        job.g = g;
        job.s_int.resize((size_t)ks[i]);
        for (int32_t s = 0; s < ks[i]; ++s) job.s_int[(size_t)s] = g->h_perm[(size_t)sources[i][s]];
        job.reqs.push_back({0, ks[i], outs[i]});
        jobs.push_back(std::move(job));
        at.push_back(i);
    }
    std::vector<char> over;
    const bc_status st = source_jobs(jobs, stream, over);
    const bool no_room = st == BC_ERR_OUT_OF_MEMORY;  // the host loop may have some
    if (no_room) (void)hipGetLastError();
    else if (st != BC_OK) return st;
    for (size_t j = 0; j < at.size(); ++j) {
        if (!no_room && !over[j]) continue;
        if (!no_room) range_exceeded(gs[at[j]]);
        alone.push_back(at[j]);
    }
    std::sort(alone.begin(), alone.end());
    for (int32_t i = 0; loops && i < ng; ++i) loops[i] = BC_LOOP_DEVICE;
    bool range = false;
    for (int32_t i : alone) {
        bc_graph_s *g = gs[i];
        if (loops) loops[i] = BC_LOOP_HOST;
        const bc_status s2 = batched_run(g, sources[i], ks[i], outs[i], kWave,
                                         g->tuned_sparse_div.load(), 0, BC_LOOP_HOST, stream,
                                         nullptr, nullptr);
        if (s2 == BC_ERR_RANGE) range = true;
        else if (s2 != BC_OK) return s2;
    }
    return range ? BC_ERR_RANGE : BC_OK;
}

// Batches run at once for `concurrency` (0: by workspace size; the choice
// depends only on the graph and the batch count, so results are identical
// from run to run).  Parts overlap one another's small kernels and host
// polls; beyond the process's 4 hardware queues they gain nothing, and the
// large graphs' level kernels already fill the device.
int32_t parts_of(const bc_graph_s *g, int32_t concurrency, int32_t nbatches, int32_t H) {
    int32_t p = concurrency;
    if (p <= 0) {
        const size_t ws = batch_ws_bytes(g, H) + batch_level_bytes(g, 16, H);
        p = ws <= ((size_t)1 << 30) ? 4 : (ws <= ((size_t)16 << 30) ? 2 : 1);
    }
    return std::max(1, std::min(p, nbatches));
}

bc_status get_streams(bc_graph_s *g, int32_t p, std::vector<hipStream_t> &out) {
    std::lock_guard<std::mutex> lk(g->stream_mu);
    while ((int32_t)g->streams.size() < p) {
        hipStream_t st = nullptr;
        BC_TRY_HIP(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
        g->streams.push_back(st);
    }
    out.assign(g->streams.begin(), g->streams.begin() + p);
    return BC_OK;
}

// Batch composition: sources sorted by their distances to the two landmarks,
// so that the sources of a batch lie close together and see most vertices at
// the same level (their frontier masks share lanes, the row gathers are
// dense).  BC is a sum over sources, so any grouping gives the same result up
// to rounding; the order depends only on the inputs.  order[i] = caller index
// of lane i of the run, s_int = its internal source ids, plan = batches of
// `width` lanes.
bc_status make_plan(bc_graph_s *g, const int32_t *sources, int32_t k, int32_t width,
                    std::vector<int32_t> &order, std::vector<int32_t> &s_int,
                    std::vector<BatchPlan> &plan) {
    order.assign((size_t)k, 0);
    for (int32_t i = 0; i < k; ++i) order[(size_t)i] = i;
    if (k > width && !g->directed) {  // the landmarks' BFS runs undirected
        bc_status st = ensure_landmarks(g);
        if (st != BC_OK) return st;
        const uint32_t far = 0x7fffffff;
        auto key = [&](int32_t i) {
            const int32_t v = g->h_perm[(size_t)sources[i]];
            const int32_t a = g->land1[(size_t)v], b = g->land2[(size_t)v];
            return std::make_pair(a < 0 ? far : (uint32_t)a, b < 0 ? far : (uint32_t)b);
        };
        std::stable_sort(order.begin(), order.end(),
                         [&](int32_t x, int32_t y) { return key(x) < key(y); });
    }
    s_int.assign((size_t)k, 0);
    for (int32_t i = 0; i < k; ++i) s_int[(size_t)i] = g->h_perm[(size_t)sources[order[(size_t)i]]];
    plan.clear();
    for (int32_t b0 = 0; b0 < k; b0 += width) plan.push_back({b0, std::min(width, k - b0), 0, 0});
    return BC_OK;
}

bc_status batched_run(bc_graph_s *g, const int32_t *sources, int32_t k, double *bc_out,
                      int32_t width, int32_t sparse_div, int32_t concurrency,
                      int32_t level_loop, hipStream_t stream, int32_t *dist, double *sigma) {
    if (use_source(g, level_loop, k, width)) {
        std::vector<SourceJob> jobs(1);
        SourceJob &job = jobs[0];
        job.g = g;
        job.s_int.resize((size_t)k);
        std::vector<int32_t> rows((size_t)k);
        for (int32_t i = 0; i < k; ++i) {
            job.s_int[(size_t)i] = g->h_perm[(size_t)sources[i]];
            rows[(size_t)i] = i;
        }
        job.reqs.push_back({0, k, bc_out});
        if (dist || sigma) {
            job.export_row = rows.data();
            job.dist = dist;
            job.sigma = sigma;
            const size_t cells = (size_t)k * (size_t)g->n;
            if (dist) BC_TRY_HIP(hipMemsetAsync(dist, 0xff, cells * sizeof(int32_t), stream));
            if (sigma) BC_TRY_HIP(hipMemsetAsync(sigma, 0, cells * sizeof(double), stream));
        }
        std::vector<char> over;
        const bc_status st = source_jobs(jobs, stream, over);
        // a count beyond double's range sends the call to the host loop, as
        // does scratch that does not fit
        if (st == BC_ERR_OUT_OF_MEMORY) (void)hipGetLastError();
        else if (st != BC_OK || !over[0]) return st;
        else range_exceeded(g);
    }
    const bool state = dist || sigma;  // per-source exports: not on the pair path
    if (!state && use_pair(g, level_loop, width)) {
        bc_status st = pair_run(g, sources, k, bc_out, stream);
        if (st != BC_ERR_OUT_OF_MEMORY) return st;
        // no room for the queues: what a graph that is not deep takes
        (void)hipGetLastError();
        (void)bc_trim_workspaces(g);
        if (k < g->tuned_min_batched.load() && !g->sigma_ext.load()) {
            st = plain_run(g, sources, k, bc_out, nullptr, stream, nullptr, nullptr);
            if (st != BC_ERR_RANGE) return st;
            range_exceeded(g);
        }
    }
    std::vector<int32_t> order, s_int;
    std::vector<BatchPlan> plan;
    {
        const bc_status st0 = make_plan(g, sources, k, width, order, s_int, plan);
        if (st0 != BC_OK) return st0;
    }
    const int32_t P = parts_of(g, concurrency, (int32_t)plan.size(), width > kWave ? 2 : 1);
    if (P <= 1)
        return run_batch_plan(g, s_int, plan, {}, {}, bc_out, stream, order.data(), dist, sigma,
                              sparse_div, level_loop == BC_LOOP_GRAPH);
    // P parts of consecutive batches, each on its own stream and workspace,
    // ordered after the caller's earlier work; BC = the parts' sum in part
    // order, on the caller's stream
    std::vector<hipStream_t> streams;
    bc_status st = get_streams(g, P, streams);
    if (st != BC_OK) return st;
    const size_t n = (size_t)g->n;
    double *parts = nullptr;
    hipEvent_t ev_start = nullptr;
    std::vector<hipEvent_t> ev_done((size_t)P, nullptr);
    auto cleanup = [&]() {
        if (parts) (void)hipFree(parts);
        if (ev_start) (void)hipEventDestroy(ev_start);
        for (hipEvent_t ev : ev_done)
            if (ev) (void)hipEventDestroy(ev);
    };
    hipError_t e = hipMalloc(&parts, (size_t)P * n * sizeof(double));
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ev_start, hipEventDisableTiming);
    for (int32_t i = 0; i < P && e == hipSuccess; ++i)
        e = hipEventCreateWithFlags(&ev_done[(size_t)i], hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(ev_start, stream);
    for (int32_t i = 0; i < P && e == hipSuccess; ++i) e = hipStreamWaitEvent(streams[i], ev_start, 0);
    if (e != hipSuccess) {
        cleanup();
        return from_hip(e);
    }
    const int32_t nb = (int32_t)plan.size();
    std::vector<bc_status> status((size_t)P, BC_OK);
    std::vector<std::thread> workers;
    for (int32_t i = 0; i < P; ++i) {
        workers.emplace_back([&, i]() {
            DeviceGuard dg(g->device);
            const int32_t b0 = (int32_t)((int64_t)nb * i / P), b1 = (int32_t)((int64_t)nb * (i + 1) / P);
            std::vector<BatchPlan> sub(plan.begin() + b0, plan.begin() + b1);
            status[(size_t)i] = run_batch_plan(g, s_int, sub, {}, {}, parts + (size_t)i * n,
                                               streams[(size_t)i], order.data(), dist, sigma,
                                               sparse_div, level_loop == BC_LOOP_GRAPH);
            if (hipEventRecord(ev_done[(size_t)i], streams[(size_t)i]) != hipSuccess &&
                status[(size_t)i] == BC_OK)
                status[(size_t)i] = BC_ERR_DEVICE;
        });
    }
    for (std::thread &t : workers) t.join();
    bc_status result = BC_OK;
    for (bc_status s2 : status) {
        if (s2 != BC_OK && s2 != BC_ERR_RANGE) {
            result = s2;
            break;
        }
        if (s2 == BC_ERR_RANGE) result = BC_ERR_RANGE;
    }
    for (int32_t i = 0; i < P && e == hipSuccess; ++i) e = hipStreamWaitEvent(stream, ev_done[i], 0);
    if (e == hipSuccess && (result == BC_OK || result == BC_ERR_RANGE))
        e = sum_parts(g->n, parts, P, bc_out, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    cleanup();
    if (e != hipSuccess) return from_hip(e);
    return result;
}

// Several requests in one run.  A request of at most 64 sources never
// straddles two batches; a larger one fills whole batches and its remainder
// goes like a small request.  Every request's result is then made of the same
// lanes in the same order whatever else shares its batches: the whole batches
// run first, then the shared ones, which the small requests and remainders
// fill largest first, each into the first with room (the order of arrival took
// five batches where three hold the requests 1, 8, 64, 1, 8, 64, 1, 7: 4.6
// -> 2.9 ms on the 65K-vertex R-MAT).
bc_status multi_run(bc_graph_s *g, const int32_t *sources, const int32_t *req_start,
                    int32_t nreq, double *const *outs, hipStream_t stream) {
    const int32_t k = req_start[nreq];
    std::vector<int32_t> s_int((size_t)k);
    for (int32_t i = 0; i < k; ++i) s_int[(size_t)i] = g->h_perm[(size_t)sources[i]];
    if (multi_source(g)) {
        std::vector<SourceJob> jobs(1);
        jobs[0].g = g;
        jobs[0].s_int = s_int;
        for (int32_t r = 0; r < nreq; ++r)
            jobs[0].reqs.push_back({req_start[r], req_start[r + 1] - req_start[r], outs[r]});
        std::vector<char> over;
        const bc_status st = source_jobs(jobs, stream, over);
        if (st == BC_ERR_OUT_OF_MEMORY) (void)hipGetLastError();
        else if (st != BC_OK || !over[0]) return st;
        else range_exceeded(g);  // the call runs again level-scaled
    }
    struct Share {
        int32_t req, first, lanes;  // sources [first, first + lanes) of the call
    };
    std::vector<std::vector<Share>> batches;
    std::vector<Share> small;
    for (int32_t r = 0; r < nreq; ++r) {
        int32_t at = req_start[r];
        for (; req_start[r + 1] - at >= kWave; at += kWave) batches.push_back({{r, at, kWave}});
        if (at < req_start[r + 1]) small.push_back({r, at, req_start[r + 1] - at});
    }
    std::stable_sort(small.begin(), small.end(),
                     [](const Share &x, const Share &y) { return x.lanes > y.lanes; });
    const size_t whole = batches.size();
    std::vector<int32_t> room;  // of the shared batches; by lanes, the first that may have it
    size_t from[kWave + 1] = {};
    for (const Share &sh : small) {
        size_t &b = from[sh.lanes];
        while (b < room.size() && room[b] < sh.lanes) ++b;
        if (b == room.size()) {
            room.push_back(kWave);
            batches.push_back({});
        }
        room[b] -= sh.lanes;
        batches[whole + b].push_back(sh);
    }
    std::vector<BatchPlan> plan;
    std::vector<int32_t> seg_start, lanes;
    std::vector<double *> seg_out;
    for (const std::vector<Share> &batch : batches) {
        // seg_out entries of batch b are stored at seg_first - b (one fewer
        // entry than seg_start per batch): both tables aligned by index
        BatchPlan bp{(int32_t)lanes.size(), 0, (int32_t)seg_start.size(), (int32_t)batch.size()};
        for (const Share &sh : batch) {
            seg_start.push_back(bp.nlanes);
            seg_out.push_back(outs[sh.req]);
            bp.nlanes += sh.lanes;
            lanes.insert(lanes.end(), s_int.begin() + sh.first, s_int.begin() + sh.first + sh.lanes);
        }
        seg_start.push_back(bp.nlanes);
        plan.push_back(bp);
    }
    s_int.swap(lanes);
    for (int32_t r = 0; r < nreq; ++r) {
        hipError_t e = hipMemsetAsync(outs[r], 0, (size_t)g->n * sizeof(double), stream);
        if (e != hipSuccess) return from_hip(e);
    }
    return run_batch_plan(g, s_int, plan, seg_start, seg_out, nullptr, stream, nullptr, nullptr,
                          nullptr, g->tuned_sparse_div.load(), false);
}

}  // namespace bcx
