// Brandes betweenness centrality with one workgroup per source, for graphs
// whose per-source state fits a compute unit's LDS.
//
// The computation is the paper's (Section "Background", the ComputeBC
// listing): a forward breadth-first pass summing sigma over parents, then a
// reverse pass over the levels summing dependencies over children.  A
// workgroup of 16 waves runs a whole source, every level, with workgroup
// barriers between levels, so a call is one launch whatever its depth, and
// 256 compute units work on different sources without sharing anything.
//
// State of a source:
//   val    a double per vertex in LDS.  Forward: kUnreached (a NaN), 0 once
//          claimed for a level, then +sigma on even levels and -sigma on odd
//          ones.  Reverse: 0, then +-c (c = (1 + delta) / sigma) by the same
//          parity.  A vertex at level L sums max(+-val, 0) over its arcs,
//          with the sign of the level it pulls from: everything that is not a
//          parent (child) adds 0.  Neighbours lie within one level of each
//          other, except that a directed arc may lead back to any earlier
//          level: those still hold 0 in the reverse pass, and no arc into v
//          comes from a level before L-1 in the forward one.  So an arc costs
//          its id, one LDS double, a max and an add, with no level array and
//          no branch.
//   queue  every level back to back (global), one per degree class: vertices
//          of more than 512 arcs take a wave each, of 65 .. 512 arcs 16
//          lanes, of 9 .. 64 arcs 4 lanes, of up to 8 arcs one lane.
//   sig    sigma in queue order (global), for the reverse pass.
// Larger graphs (kMem) keep val in memory, where 0 takes the place of both
// sentinels, and in LDS a bit per vertex for the claims and one for the queued.
// A vertex's sums run over its arcs in a fixed order (each lane its arcs in
// turn, then a butterfly), whatever order the queue has, so results repeat
// bit for bit.
//
// What bounds it: instruction issue.  A turn of 256 arcs costs some 40 vector
// instructions and a task 100 more (queue entry, row bounds, the sum over its
// lanes, a division), so the classes give a task 4 to 64 vertices; a first
// version with a level code per vertex, a branch per DAG arc and an append
// per claim took 0.58 ms where this one takes 0.28 (R-MAT of 16K vertices,
// edge factor 16, 64 sources).  Measured against one workgroup per batch of
// 64 sources (64-value rows in global memory): all sources of the 4K-vertex
// R-MAT (edge factor 8) 4.48 -> 0.71 ms, 16 graphs of 1K to 4K vertices with
// 64 sources each in one call 5.75 -> 0.26 ms; against the one-source path,
// one source of the 4K-vertex R-MAT 0.173 -> 0.084 ms.  With the values in
// memory it is bound by their lines in the L2 (a compute unit's 8 n bytes, 32
// units to a 4 MB L2): 16,384 sources on 21K vertices of 4 arcs each take 24.4
// ms, the host loop 160; of the 33K-vertex R-MAT (edge factor 4) 26.8 and 80.4;
// 32 graphs of 30K vertices, 64 sources each in one call, 6.6 and 42.9.  (One
// workgroup per 64-source batch, as these graphs once ran: 52, 52.5 and 32.8.)
#include "bc_internal.h"
#include "bc_wave.h"

namespace bcx {
namespace {

constexpr int kSrcBlock = 1024;
constexpr int kSrcWaves = kSrcBlock / kWave;
constexpr uint32_t kUnreachedHi = 0x7ff80000u;  // high word of kUnreached (low word 0)

struct SrcWork {
    uint32_t owners = 0, arcs = 0, hits = 0;
};

// x + (x of the lane that the DPP control names), on the vector units (a
// shuffle through the LDS crossbar takes over 100 cycles, and a vertex's
// whole sum waits for six of them).
template <int kCtrl>
__device__ __forceinline__ double add_dpp(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), kCtrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), kCtrl, 0xf, 0xf, false);
    return x + __hiloint2double(hi, lo);
}

__device__ __forceinline__ double read_lane(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Sum over the W lanes of a vertex, pairwise in the order of a butterfly.
template <int W>
__device__ __forceinline__ double lanes_sum(double x) {
    static_assert(W == 1 || W == 4 || W == 16 || W == kWave, "lanes per vertex");
    if (W == 1) return x;
    BC_FULL_EXEC();
    x = add_dpp<0xB1>(x);   // quad_perm 1,0,3,2: lane ^ 1
    x = add_dpp<0x4E>(x);   // quad_perm 2,3,0,1: lane ^ 2
    if (W == 4) return x;
    x = add_dpp<0x141>(x);  // row_half_mirror: the other four of each eight
    x = add_dpp<0x140>(x);  // row_mirror: the other eight of each sixteen
    if (W == 16) return x;
    return (read_lane(x, 0) + read_lane(x, 16)) + (read_lane(x, 32) + read_lane(x, 48));
}

// A value that is the same in every lane, held in scalar registers.
__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }

template <typename T> __device__ __forceinline__ T *uniform(T *p) {
    const uint64_t x = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)uniform((int32_t)(uint32_t)x);
    const uint32_t hi = (uint32_t)uniform((int32_t)(uint32_t)(x >> 32));
    return reinterpret_cast<T *>(((uint64_t)hi << 32) | lo);
}

// What a source's pass works on (every field uniform).
struct SrcView {
    int32_t n;
    int32_t c1, c2, c3;   // class c's ids and queue start at 0, c1, c2, c3
    const int32_t *row_ptr, *col_idx, *row_ptr_in, *col_idx_in;
    double *val;          // [n + 1], entry n always 0; in LDS but with kMem
    uint32_t *seen, *done;  // kMem: bits in LDS of the vertices claimed, of those queued
    int32_t *q;           // [n]: the classes' queues
    double *sig;          // [n]: sigma, in queue order
    __device__ __forceinline__ int32_t base(int c) const {
        return c == 0 ? 0 : (c == 1 ? c1 : (c == 2 ? c2 : c3));
    }
    __device__ __forceinline__ int32_t past(int c) const {
        return c == 0 ? c1 : (c == 1 ? c2 : (c == 2 ? c3 : n));
    }
};

// A vertex's value: with kMem the sentinel for one not claimed in the forward
// pass (kFwd), whose memory holds 0.
template <bool kMem, bool kFwd>
__device__ __forceinline__ double value_of(const SrcView &s, int32_t id) {
    if (kMem && kFwd && !((s.seen[id >> 5] >> (id & 31)) & 1u))
        return __hiloint2double((int)kUnreachedHi, 0);
    return s.val[id];
}

// Builds the queues of level L+1 from the vertices that level L claimed, the
// ones whose value is 0: 64 ids per wave and turn, their places in the queues
// taken with one LDS atomic per class among them.  `start`: the level's queue
// positions, cnt_next: its counts so far.  The scan of n LDS words costs less
// than a queue append per claim: a claim is then a plain store, and the queue
// comes out in id order, neighbouring rows beside each other.
template <bool kMem>
__device__ __forceinline__ void collect(const SrcView &s, uint32_t *cnt_next,
                                        const uint32_t (&start)[kSrcClasses]) {
    BC_FULL_EXEC();
    const int lane = lane_id();
    if constexpr (kMem) {  // the claims are 32 to a word, a word per lane
        const int32_t words = (s.n + 32) / 32;
        for (int32_t w0 = (int32_t)(threadIdx.x & ~(kWave - 1u)); w0 < words; w0 += kSrcBlock) {
            const int32_t w = w0 + lane;
            uint32_t got = 0;
            if (w < words) {
                const uint32_t now = s.seen[w];
                got = now & ~s.done[w];
                s.done[w] = now;
            }
            if (__ballot(got != 0u) == 0ull) continue;
#pragma unroll
            for (int c = 0; c < kSrcClasses; ++c) {
                if (s.past(c) <= 32 * w0 || s.base(c) >= 32 * (w0 + kWave)) continue;
                const int32_t b = s.base(c) - 32 * w, e = s.past(c) - 32 * w;
                uint32_t m = got;  // ... those of the class: bits [b, e)
                if (b > 0) m = b < 32 ? m & (~0u << b) : 0u;
                if (e < 32) m = e > 0 ? m & ~(~0u << e) : 0u;
                if (__ballot(m != 0u) == 0ull) continue;
                uint32_t total;
                const uint32_t mine = wave_excl_scan((uint32_t)__popc(m), total);
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&cnt_next[c], total);
                at = (uint32_t)uniform((int32_t)at) + (uint32_t)s.base(c) + start[c] + mine;
                for (; m; m &= m - 1u) s.q[at++] = 32 * w + __builtin_ctz(m);
            }
        }
        return;
    }
    for (int32_t v0 = (int32_t)(threadIdx.x & ~(kWave - 1u)); v0 < s.n; v0 += kSrcBlock) {
        const int32_t v = v0 + lane;
        const bool got = v < s.n && __double2hiint(s.val[v]) == 0;
        if (__ballot(got) == 0ull) continue;
#pragma unroll
        for (int c = 0; c < kSrcClasses; ++c) {
            if (s.past(c) <= v0 || s.base(c) >= v0 + kWave) continue;
            const uint64_t m = __ballot(got && v >= s.base(c) && v < s.past(c));
            if (m == 0ull) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&cnt_next[c], (uint32_t)__popcll(m));
            at = (uint32_t)uniform((int32_t)at) + (uint32_t)s.base(c) + start[c];
            if ((m >> lane) & 1ull)
                s.q[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = v;
        }
    }
}

// Four consecutive arc ids, loaded at once (rows start at any arc, so the
// address is only 4-byte aligned; the arrays end in kArcPad spare ids).
struct __attribute__((packed, aligned(4))) Ids {
    int32_t id[4];
};
static_assert(kArcPad >= 3, "a load of four ids may pass the last arc by three");

// This lane's share of an adjacency row: four arcs from e, the next four
// 4 W further on, below re.
struct Row {
    int32_t e = 0, re = 0;
};

__device__ __forceinline__ Row row_of(const int32_t *rp, int32_t v, int sl) {
    Row r;
    if (v >= 0) {
        r.e = rp[v] + 4 * sl;
        r.re = rp[v + 1];
    }
    return r;
}

__device__ __forceinline__ Ids ids_at(const int32_t *col, Row r) {
    Ids x = {{0, 0, 0, 0}};
    // (a 32-bit byte offset: the library takes this path below 2^30 arcs)
    if (r.e < r.re)
        x = *reinterpret_cast<const Ids *>(reinterpret_cast<const char *>(col) +
                                           (uint32_t)r.e * 4u);
    return x;
}

// Calls body(ids, values) for every four arcs of each lane's row, the next
// four ids already on their way (W lanes per vertex; slots past the row's end
// get id n, whose value is 0).
template <int W, bool kMem, bool kFwd, typename Body>
__device__ __forceinline__ void over_row(const SrcView &s, const int32_t *col, Row r,
                                         Body &&body) {
    Ids nx = ids_at(col, r);
    while (__ballot(r.e < r.re)) {
        BC_FULL_EXEC();
        Ids x = nx;
        const int left = r.re - r.e;
        r.e += 4 * W;
        nx = ids_at(col, r);
        double y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x.id[u] = u < left ? x.id[u] : s.n;
#pragma unroll
        for (int u = 0; u < 4; ++u) y[u] = value_of<kMem, kFwd>(s, x.id[u]);
        body(x, y);
    }
}

// A wave's task: a vertex per W lanes (v = -1: none), its queue position and
// its rows.
struct Task {
    int32_t v = -1;
    uint32_t at = 0;
    double sig = 1.0;
    Row out, in;
};

// Adds the four values pulled, those of sign `sign` (+1 or -1).
template <bool kStat>
__device__ __forceinline__ void pull4(const SrcView &s, const Ids &x, const double (&y)[4],
                                      double sign, double &acc, SrcWork &wk) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const double z = fmax(sign * y[u], 0.0);  // (0 for kUnreached too)
        acc += z;
        if (kStat) {
            wk.arcs += x.id[u] != s.n ? 1u : 0u;
            wk.hits += z > 0.0 ? 1u : 0u;
        }
    }
}

// Claims the unreached ones of four neighbours for level L+1 (NaN -> 0 by its
// high word; every claimer stores the same; with kMem, their bits).
template <bool kMem>
__device__ __forceinline__ void push4(const SrcView &s, const Ids &x, const double (&y)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if ((uint32_t)__double2hiint(y[u]) == kUnreachedHi) {
            if (kMem) atomicOr(&s.seen[x.id[u] >> 5], 1u << (x.id[u] & 31));
            else *(reinterpret_cast<volatile uint32_t *>(&s.val[x.id[u]]) + 1) = 0u;
        }
}

// Forward step of one vertex per W lanes: sigma over the arcs into it from
// level L-1 (sign `par`), unreached neighbours claimed for level L+1.
// Undirected graphs read each adjacency row once for both.
template <int W, bool kDir, bool kMem, bool kStat>
__device__ __forceinline__ void fwd_vertex(const SrcView &s, const Task &k, bool source,
                                           double par, int32_t *range, SrcWork &wk) {
    double acc = 0.0;
    if (kDir) {
        over_row<W, kMem, true>(s, s.col_idx_in, k.in,
                    [&](const Ids &x, const double (&y)[4]) __attribute__((always_inline)) {
                        pull4<kStat>(s, x, y, par, acc, wk);
                    });
        over_row<W, kMem, true>(s, s.col_idx, k.out,
                    [&](const Ids &x, const double (&y)[4]) __attribute__((always_inline)) {
                        push4<kMem>(s, x, y);
                    });
    } else {
        over_row<W, kMem, true>(s, s.col_idx, k.out,
                    [&](const Ids &x, const double (&y)[4]) __attribute__((always_inline)) {
                        pull4<kStat>(s, x, y, par, acc, wk);
                        push4<kMem>(s, x, y);
                    });
    }
    acc = lanes_sum<W>(acc);
    if (k.v >= 0 && (lane_id() & (W - 1)) == 0) {
        if (source) acc = 1.0;
        s.val[k.v] = -par * acc;
        s.sig[k.at] = acc;
        if (!(acc <= 0x1.fffffffffffffp+1023)) *range = 1;
        if (kStat) ++wk.owners;
    }
}

// Reverse step of one vertex per W lanes: the children's c summed (sign
// `child`; no arcs are passed at the deepest level), delta = sigma * sum
// added to the unit's BC row.
template <int W, bool kMem, bool kStat>
__device__ __forceinline__ void bwd_vertex(const SrcView &s, const Task &k, double child,
                                           double *row, bool first, SrcWork &wk) {
    double acc = 0.0;
    over_row<W, kMem, false>(s, s.col_idx, k.out,
                [&](const Ids &x, const double (&y)[4]) __attribute__((always_inline)) {
                    pull4<kStat>(s, x, y, child, acc, wk);
                });
    acc = lanes_sum<W>(acc);
    if (k.v >= 0 && (lane_id() & (W - 1)) == 0) {
        const double delta = k.sig * acc;
        s.val[k.v] = -child * ((1.0 + delta) / k.sig);
        // one add per vertex and source, so the order is the sources'; the
        // add is left to the cache, as a load here would stall the wave
        if (delta != 0.0) {
            if (first) row[k.v] = delta;
            else unsafeAtomicAdd(&row[k.v], delta);
        }
        if (kStat) ++wk.owners;
    }
}

// Lanes per vertex of class c, as a shift.
__device__ __forceinline__ int lane_shift(int c) { return c == 0 ? 6 : (c == 1 ? 4 : (c == 2 ? 2 : 0)); }

// Runs `step(class, task)` over a level's vertices, queue positions [lo, hi)
// per class: the classes' wave tasks back to back, dealt to the waves in
// turn.  A task's vertices are loaded two tasks ahead and its row bounds (and
// sigmas) one ahead, so it waits for its arcs' ids only.
template <bool kOut, bool kIn, bool kSig, typename Step>
__device__ __forceinline__ void over_level(const SrcView &s, const uint32_t (&lo)[kSrcClasses],
                                           const uint32_t (&hi)[kSrcClasses], Step &&step) {
    const int lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t end[kSrcClasses];  // past the class's last task
#pragma unroll
    for (int c = 0; c < kSrcClasses; ++c) {
        const int per = 6 - lane_shift(c);  // vertices per task, as a shift
        end[c] = (c ? end[c - 1] : 0u) + ((hi[c] - lo[c] + (1u << per) - 1u) >> per);
    }
    const uint32_t tasks = end[kSrcClasses - 1];
    if (wave >= tasks) return;
    auto cls = [&](uint32_t t) { return t < end[0] ? 0 : (t < end[1] ? 1 : (t < end[2] ? 2 : 3)); };
    auto vertex = [&](uint32_t t, Task &k) {
        const int c = cls(t);
        const uint32_t t0 = c == 0 ? 0u : (c == 1 ? end[0] : (c == 2 ? end[1] : end[2]));
        const uint32_t l0 = c == 0 ? lo[0] : (c == 1 ? lo[1] : (c == 2 ? lo[2] : lo[3]));
        const uint32_t h0 = c == 0 ? hi[0] : (c == 1 ? hi[1] : (c == 2 ? hi[2] : hi[3]));
        const int sh = lane_shift(c);
        const uint32_t i = l0 + ((t - t0) << (6 - sh)) + (uint32_t)(lane >> sh);
        k.v = -1;
        k.at = (uint32_t)s.base(c) + i;
        if (t < tasks && i < h0) k.v = s.q[k.at];
    };
    auto rows = [&](uint32_t t, Task &k) {
        const int sl = lane & ((1 << lane_shift(cls(t))) - 1);
        if (kOut) k.out = row_of(s.row_ptr, k.v, sl);
        if (kIn) k.in = row_of(s.row_ptr_in, k.v, sl);
        if (kSig && k.v >= 0) k.sig = s.sig[k.at];
    };
    Task k0, k1;
    vertex(wave, k0);
    vertex(wave + kSrcWaves, k1);
    rows(wave, k0);
    for (uint32_t t = wave; t < tasks; t += kSrcWaves) {
        Task k2;
        vertex(t + 2 * kSrcWaves, k2);
        rows(t + kSrcWaves, k1);
        step(cls(t), k0);
        k0 = k1;
        k1.v = k2.v;
        k1.at = k2.at;
    }
}

// One workgroup per unit: the unit's sources one after another, their
// dependencies added to the unit's BC row in that order.
template <bool kDir, bool kMem, bool kStat>
__global__ __launch_bounds__(kSrcBlock, 8) void
k_source(const SourceUnit *units, const SourceGraph *graphs, const int32_t *sources,
         int32_t *range_flags, unsigned long long *stats) {
    extern __shared__ double lds[];
    __shared__ uint32_t cnt[3][kSrcClasses];
    const SourceUnit &un = units[blockIdx.x];
    const int32_t gi = uniform(un.graph);
    int32_t *range = range_flags + gi;
    SrcView s;
    const int32_t n = uniform(graphs[gi].n);
    s.n = n;
    s.c1 = uniform(graphs[gi].cls[1]);
    s.c2 = uniform(graphs[gi].cls[2]);
    s.c3 = uniform(graphs[gi].cls[3]);
    s.row_ptr = uniform(graphs[gi].row_ptr);
    s.col_idx = uniform(graphs[gi].col_idx);
    s.row_ptr_in = uniform(graphs[gi].row_ptr_in);
    s.col_idx_in = uniform(graphs[gi].col_idx_in);
    const int32_t words = (n + 32) / 32;  // bits of the vertices and of entry n
    s.seen = reinterpret_cast<uint32_t *>(lds);
    s.done = s.seen + words;
    s.q = uniform(un.q);
    s.sig = uniform(un.sig);
    if constexpr (kMem) s.val = s.sig + source_val(n);
    else s.val = lds;
    double *row = uniform(un.row);
    uint32_t *lvl = uniform(un.lvl);
    const int32_t first = uniform(un.first), count = uniform(un.count);
    // (read once: the tables are in host memory)
    int32_t *dist = uniform(un.dist);
    double *sigma = uniform(un.sigma), *out = uniform(un.out);
    const int t = threadIdx.x;
    SrcWork wf, wb;
    uint32_t verts = 0;
    int32_t depth_sum = 0;
    for (int32_t v = t; v < n; v += kSrcBlock) row[v] = 0.0;
    for (int32_t i = 0; i < count; ++i) {
        const int32_t src = uniform(sources[first + i]);
        const double unreached = kMem ? 0.0 : __hiloint2double((int)kUnreachedHi, 0);
        for (int32_t v = t; v <= n; v += kSrcBlock)
            s.val[v] = v == src || v == n ? 0.0 : unreached;
        if (kMem)
            for (int32_t w = t; w < words; w += kSrcBlock) {
                const uint32_t x = (w == src >> 5 ? 1u << (src & 31) : 0u) |
                                   (w == n >> 5 ? 1u << (n & 31) : 0u);
                s.seen[w] = x;
                s.done[w] = x;
            }
        if (t < 3 * kSrcClasses) (&cnt[0][0])[t] = 0;
        int sc = 0;
        int32_t q0 = 0;
#pragma unroll
        for (int c = 1; c < kSrcClasses; ++c)
            if (src >= s.base(c)) {
                sc = c;
                q0 = s.base(c);
            }
        if (t == 0) s.q[q0] = src;
        __syncthreads();
        // forward: lo / hi are level L's queue positions per class; level
        // L+1's vertices are counted in set (L+1) % 3, which a thread cleared
        // two levels ago (after every wave had read it)
        uint32_t lo[kSrcClasses], hi[kSrcClasses];
#pragma unroll
        for (int c = 0; c < kSrcClasses; ++c) {
            lo[c] = 0;
            hi[c] = c == sc ? 1u : 0u;
        }
        int32_t L = 0;
        for (;;) {
            if (t < kSrcClasses) {
                cnt[(L + 2) % 3][t] = 0;
                lvl[(size_t)L * kSrcClasses + t] =
                    t == 0 ? lo[0] : (t == 1 ? lo[1] : (t == 2 ? lo[2] : lo[3]));
            }
            uint32_t *cn = cnt[(L + 1) % 3];
            const double par = (L & 1) ? 1.0 : -1.0;  // sign of level L-1
            over_level<true, kDir, false>(s, lo, hi, [&](int cls, const Task &k)
                                          __attribute__((always_inline)) {
                if (cls == 0) fwd_vertex<kWave, kDir, kMem, kStat>(s, k, L == 0, par, range, wf);
                else if (cls == 1) fwd_vertex<16, kDir, kMem, kStat>(s, k, L == 0, par, range, wf);
                else if (cls == 2) fwd_vertex<4, kDir, kMem, kStat>(s, k, L == 0, par, range, wf);
                else fwd_vertex<1, kDir, kMem, kStat>(s, k, L == 0, par, range, wf);
            });
            __syncthreads();
            collect<kMem>(s, cn, hi);
            __syncthreads();
            uint32_t found = 0;
#pragma unroll
            for (int c = 0; c < kSrcClasses; ++c) {
                const uint32_t k = (uint32_t)uniform((int32_t)cn[c]);
                lo[c] = hi[c];
                hi[c] += k;
                found += k;
            }
            if (found == 0) break;
            ++L;
        }
        const int32_t deepest = L;
        depth_sum += deepest;
        if (dist || sigma) {  // (hi: the end of every queue)
            const size_t at = (size_t)un.export_row[i] * (size_t)n;
            const int32_t *iperm = graphs[gi].iperm;
            for (int32_t x = 0; x <= deepest; ++x)
#pragma unroll
                for (int c = 0; c < kSrcClasses; ++c) {
                    const uint32_t a = lvl[(size_t)x * kSrcClasses + c];
                    const uint32_t b = x < deepest ? lvl[(size_t)(x + 1) * kSrcClasses + c] : hi[c];
                    for (uint32_t p = a + t; p < b; p += kSrcBlock) {
                        const int32_t o = iperm[s.q[s.base(c) + p]];
                        if (dist) dist[at + o] = x;
                        if (sigma) sigma[at + o] = s.sig[s.base(c) + p];
                    }
                }
        }
        // reverse: levels deepest .. 1
        for (int32_t v = t; v < n; v += kSrcBlock) s.val[v] = 0.0;
        uint32_t end[kSrcClasses];
#pragma unroll
        for (int c = 0; c < kSrcClasses; ++c) {
            end[c] = hi[c];
            lo[c] = (uint32_t)uniform((int32_t)lvl[(size_t)deepest * kSrcClasses + c]);
        }
        __syncthreads();
        for (int32_t x = deepest; x >= 1; --x) {
            uint32_t prev[kSrcClasses];  // level x-1's start, loaded ahead
#pragma unroll
            for (int c = 0; c < kSrcClasses; ++c) prev[c] = lvl[(size_t)(x - 1) * kSrcClasses + c];
            const double child = (x & 1) ? 1.0 : -1.0;  // sign of level x+1
            auto settle = [&](int cls, const Task &k) __attribute__((always_inline)) {
                if (cls == 0) bwd_vertex<kWave, kMem, kStat>(s, k, child, row, i == 0, wb);
                else if (cls == 1) bwd_vertex<16, kMem, kStat>(s, k, child, row, i == 0, wb);
                else if (cls == 2) bwd_vertex<4, kMem, kStat>(s, k, child, row, i == 0, wb);
                else bwd_vertex<1, kMem, kStat>(s, k, child, row, i == 0, wb);
            };
            if (x == deepest) over_level<false, false, true>(s, lo, end, settle);
            else over_level<true, false, true>(s, lo, end, settle);
            __syncthreads();
#pragma unroll
            for (int c = 0; c < kSrcClasses; ++c) {
                end[c] = lo[c];
                lo[c] = (uint32_t)uniform((int32_t)prev[c]);
            }
        }
        if (kStat && t == 0) verts += hi[0] + hi[1] + hi[2] + hi[3];
        __syncthreads();  // the values and queues are rewritten by the next source
    }
    if (out) {  // a request of one unit: its BC in caller order
        const int32_t *perm = uniform(graphs[gi].perm);
        for (int32_t o = t; o < n; o += kSrcBlock) out[o] = row[perm[o]];
    }
    if (kStat) {
        unsigned long long x[8] = {wf.owners, wf.arcs, wf.hits, wb.owners, wb.arcs, wb.hits,
                                   verts, (unsigned long long)(t == 0 ? depth_sum : 0)};
        const int slot[8] = {0, 1, 2, 6, 7, 8, 12, 14};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) x[j] += __shfl_xor(x[j], off);
            if (lane_id() == 0 && x[j]) {
                atomicAdd(&stats[slot[j]], x[j]);
                if (j == 6) atomicAdd(&stats[13], x[j]);
            }
        }
    }
}

// out[caller id] = the sum of the request's unit rows: sixteen at a time by a
// tree, the groups added in order with their rounding errors kept (Knuth's
// two-sum), since exact BC of a small graph adds 512 rows.
constexpr int kSumFlight = 16;
__global__ __launch_bounds__(kBlock) void k_source_sum(const SourceSum *sums) {
    const SourceSum r = sums[blockIdx.y];
    const int32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v >= r.n) return;
    const double *row = r.row + v;
    double s = 0.0, err = 0.0;
    for (int32_t u = 0; u < r.units; u += kSumFlight) {
        double x[kSumFlight];
#pragma unroll
        for (int j = 0; j < kSumFlight; ++j)
            x[j] = u + j < r.units ? row[(size_t)(u + j) * r.stride] : 0.0;
#pragma unroll
        for (int w = kSumFlight / 2; w >= 1; w /= 2)
#pragma unroll
            for (int j = 0; j < w; ++j) x[j] += x[j + w];
        const double t = s + x[0], b = t - s;
        err += (s - (t - b)) + (x[0] - b);
        s = t;
    }
    r.out[r.iperm[v]] = s + err;
}

}  // namespace

#ifdef BC_CHECK_EXEC
unsigned int exec_partial_source() { return exec_partial_take(); }
#endif

bool source_in_lds(int32_t n) { return ((size_t)n + 1) * sizeof(double) <= kSrcLdsBytes; }

size_t source_lds_bytes(int32_t n) {
    if (source_in_lds(n)) return ((size_t)n + 1) * sizeof(double);
    return 2 * (((size_t)n + 32) / 32) * sizeof(uint32_t);
}

hipError_t source_run(const SourceUnit *units, int32_t nunits, const SourceGraph *graphs,
                      const int32_t *sources, bool directed, bool in_lds, size_t lds, int32_t *range,
                      unsigned long long *stats, hipStream_t stream) {
    if (nunits <= 0) return hipSuccess;
    auto k = in_lds ? (directed ? (stats ? k_source<true, false, true> : k_source<true, false, false>)
                                : (stats ? k_source<false, false, true> : k_source<false, false, false>))
                    : (directed ? (stats ? k_source<true, true, true> : k_source<true, true, false>)
                                : (stats ? k_source<false, true, true> : k_source<false, true, false>));
    hipLaunchKernelGGL(k, dim3(nunits), dim3(kSrcBlock), lds, stream, units, graphs, sources,
                       range, stats);
    return hipGetLastError();
}

hipError_t source_sum(const SourceSum *sums, int32_t nsums, int32_t max_n, hipStream_t stream) {
    constexpr int32_t kMaxY = 65535;  // requests per launch (the grid's second dimension)
    hipError_t e = hipSuccess;
    for (int32_t a = 0; a < nsums && max_n > 0 && e == hipSuccess; a += kMaxY) {
        const int32_t m = nsums - a < kMaxY ? nsums - a : kMaxY;
        hipLaunchKernelGGL(k_source_sum, dim3((max_n + kBlock - 1) / kBlock, m), dim3(kBlock), 0,
                           stream, sums + a);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace bcx
