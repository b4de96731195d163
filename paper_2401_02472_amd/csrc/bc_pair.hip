// Brandes betweenness centrality on deep graphs of low degree (road-like
// networks): every level's (vertex, source) pairs from per-source queues.
//
// The computation is the paper's (Section "Background", the ComputeBC
// listing): forward, sigma summed over parents; reverse, dependencies summed
// over children.  On a deep graph the sources of a batch see a vertex at
// different levels, so the batched kernels' masks and 64-value rows carry one
// or two sources at a time and every level scans all vertices for them.  Here
// a level step touches only its frontier:
//
//   q[s]     source s's vertices in level order (each once); the forward pass
//            leaves in an entry's top four bits which of the vertex's arcs
//            lead to children (of up to four), so that the reverse pass loads
//            no others
//   code[s]  a byte per vertex: level mod 3, 3 = not reached (neighbours lie
//            within one level of each other, so this tells parent, sibling
//            and child apart)
//   val[s]   sigma on the way out, c = (1 + delta) / sigma on the way back
//   delta[s] dependencies, added over the sources in a fixed order at the end
//
// The arrays are one after another per source, in an order of the vertices
// (bc_layout.hip) in which the vertices of a ring of the graph lie close
// together: they share cache lines, in a level and from level to level.  One
// lane takes one pair and its few arcs (kPairMaxDeg at most).
// What bounds it: lines of scattered 8-byte values where levels are wide (a
// diagonal front meets about two vertices of a line, a pair moves some five
// lines in both passes: 0.18 ns per pair), the chain of dependent loads of a
// level where they are narrow.  Road-like grids of 1M vertices against the
// batched kernels: without shortcuts (1,700 levels, counts past double's
// range), 50 sources 238 -> 17.4 ms; with shortcuts (122 levels), 64 sources
// 23.9 -> 12.2 ms.
//
// Forward: a vertex is claimed by an atomic AND on its code; a workgroup
// collects its claims in LDS and takes their queue places with one atomic on
// the source's counter.  Queue order varies from run to run, sums do not:
// each runs over a vertex's arcs in row order.
#include "bc_internal.h"
#include "bc_wave.h"

namespace bcx {
namespace {

constexpr int kPairFlight = 4;  // arcs of a pair looked at together
// Counts from here on take exponents.  Below the largest double, so that
// (1 + delta) / sigma stays a normal number without them: a sum is then the
// same to the bit with exponents and without.
constexpr double kPairRange = 0x1p1000;

struct PairWork {
    uint32_t owners = 0, arcs = 0, hits = 0;
};

__device__ __forceinline__ void report_pairs(unsigned long long *stats, int base,
                                             const PairWork &wk) {
    BC_FULL_EXEC();
    unsigned long long x[3] = {wk.owners, wk.arcs, wk.hits};
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x[j] += __shfl_xor(x[j], off);
        if (lane_id() == 0 && x[j]) atomicAdd(&stats[base + j], x[j]);
    }
}

// A level's share of source s: positions [start, start + count) of its queue.
struct Segment {
    int32_t start, count;
};

__device__ __forceinline__ Segment segment(const PairDev &d, int32_t L, int32_t s) {
    return {d.lvl[(size_t)L * d.k + s], d.cnt[(size_t)L * d.k + s]};
}

// A vertex's arcs, four at a time: those of a vertex of up to four come from
// the graph's `four` table (one load where the row's bounds and ids would be
// two in a row), the others from its row, after an empty first turn.
struct Arcs {
    int32_t nb[4];
    int32_t e, re;  // the row's arcs still to come
};

__device__ __forceinline__ int4 four_of(const PairGraph &g, int32_t v) {
    return v >= 0 ? g.four[v] : make_int4(-1, -1, -1, -1);
}

// The arcs found are hidden from the optimiser's reasoning: knowing where an
// id is -1, it has run the cross-lane steps that follow (ballots, the leader
// lane's atomic) once for the lanes with an arc and once for those without.
__device__ __forceinline__ void hide(Arcs &a) {
#pragma unroll
    for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(a.nb[u]));
}

// (f: the vertex's entry of the table, which a caller may load ahead)
__device__ __forceinline__ Arcs first_arcs(const PairGraph &g, int32_t v, int4 f) {
    const bool more = f.x == kMoreArcs;
    Arcs a;
    a.nb[0] = more ? -1 : f.x;
    a.nb[1] = more ? -1 : f.y;
    a.nb[2] = more ? -1 : f.z;
    a.nb[3] = more ? -1 : f.w;
    a.e = more ? g.row_ptr[v] : 0;
    a.re = more ? g.row_ptr[v + 1] : 0;
    hide(a);
    return a;
}

__device__ __forceinline__ void next_arcs(const PairGraph &g, Arcs &a) {
#pragma unroll
    for (int u = 0; u < 4; ++u) a.nb[u] = a.e + u < a.re ? g.col_idx[a.e + u] : -1;
    a.e += 4;
    hide(a);
}

// A queue entry: the vertex, and above it the arcs that (may) lead to children.
constexpr int kMaskShift = 28;
__device__ __forceinline__ int32_t entry_vertex(int32_t x) {
    return x & ((1 << kMaskShift) - 1);
}
__device__ __forceinline__ uint32_t entry_mask(int32_t x) { return (uint32_t)x >> kMaskShift; }

// x 2^e, exact unless it leaves double's range.
__device__ __forceinline__ double scaled(double x, int32_t e) { return e ? ldexp(x, e) : x; }

// Block b of a level step works for source b mod turns(k) on the pieces
// b / turns(k), b / turns(k) + per, ... of 256 pairs of its level.  Not a multiple
// of eight, so that a source's blocks go round the XCDs: with all of them on one,
// as workgroups are dealt, an XCD waits for the sources whose levels are wide (ms
// per source, 1M-vertex grid with shortcuts: 63 or 65 sources 0.191, 64 0.224; 4M
// vertices 31 or 33 0.74, 32 0.91).
__host__ __device__ inline int32_t turns(int32_t k) { return k % 8 == 0 ? k + 1 : k; }

// Forward step of level L.
template <bool kExt>
__global__ __launch_bounds__(kBlock) void k_pair_forward(PairDev d, int32_t L, int32_t per) {
    __shared__ int32_t found[kBlock * kPairMaxDeg];
    __shared__ int32_t nfound, place;
    const int32_t s = (int32_t)(blockIdx.x % (uint32_t)turns(d.k));
    const int32_t piece = (int32_t)(blockIdx.x / (uint32_t)turns(d.k));
    if (s >= d.k) return;
    const Segment sg = segment(d, L, s);
    const int t = threadIdx.x;
    if (piece == 0 && t == 0) {
        d.lvl[(size_t)(L + 1) * d.k + s] = sg.start + sg.count;
        if (sg.count > 0) d.depth[s] = L;
    }
    if (piece * kBlock >= sg.count) return;
    const int par = (L + 2) % 3, nxt = (L + 1) % 3;
    int32_t *q = d.q + (size_t)s * d.stride;
    uint8_t *code = d.code + (size_t)s * d.stride;
    double *val = d.val + (size_t)s * d.stride;
    int32_t *ex = kExt ? d.ex + (size_t)s * d.stride : nullptr;
    PairWork wk;
    for (int32_t i0 = piece * kBlock; i0 < sg.count; i0 += per * kBlock) {
        if (t == 0) nfound = 0;
        __syncthreads();
        const int32_t i = i0 + t;
        const int32_t v = i < sg.count ? q[sg.start + i] : -1;
        Arcs a = first_arcs(d.g, v, four_of(d.g, v));
        double acc = 0.0;
        int32_t E = 0;  // extended range: the sum's exponent
        uint32_t mask = 0;
        for (bool first = true;; first = false) {
            const int32_t (&nb)[4] = a.nb;
            int c[kPairFlight];
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u) c[u] = nb[u] >= 0 ? code[nb[u]] : -1;
            if (first) {
#pragma unroll
                for (int u = 0; u < kPairFlight; ++u)
                    mask |= (c[u] == 3 || c[u] == nxt) ? 1u << u : 0u;
            }
            double x[kPairFlight];
            int32_t xe[kPairFlight];
            bool got[kPairFlight];
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u) {
                x[u] = 0.0;
                xe[u] = 0;
                if (c[u] == par) {
                    x[u] = val[nb[u]];
                    if (kExt) xe[u] = ex[nb[u]];
                }
                got[u] = false;
                if (c[u] == 3) {
                    const int sh = (nb[u] & 3) * 8;
                    const uint32_t old = atomicAnd(reinterpret_cast<uint32_t *>(code) + (nb[u] >> 2),
                                                   ~((uint32_t)(3 ^ nxt) << sh));
                    got[u] = ((old >> sh) & 3u) == 3u;
                }
            }
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u) {
                if (kExt) {
                    if (x[u] != 0.0) {  // to the larger exponent of the two
                        if (acc == 0.0) E = xe[u];
                        const int32_t top = E > xe[u] ? E : xe[u];
                        acc = scaled(acc, E - top) + scaled(x[u], xe[u] - top);
                        E = top;
                    }
                } else {
                    acc += x[u];
                }
                wk.arcs += nb[u] >= 0 ? 1u : 0u;
                wk.hits += c[u] == par ? 1u : 0u;
            }
            // claims in the order of the lanes, so that the queue keeps the
            // order along the rings (a list per arc slot would cut it into
            // four after each level)
            BC_FULL_EXEC();
            uint64_t m[kPairFlight], any = 0;
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u) {
                m[u] = __ballot(got[u]);
                any |= m[u];
            }
            if (any) {
                int32_t all = 0, mine = 0;
#pragma unroll
                for (int u = 0; u < kPairFlight; ++u) {
                    all += (int32_t)__popcll(m[u]);
                    mine = (int32_t)__builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(m[u] >> 32),
                        __builtin_amdgcn_mbcnt_lo((uint32_t)m[u], (uint32_t)mine));
                }
                int32_t at = 0;
                if (lane_id() == 0) at = atomicAdd(&nfound, all);
                mine += __builtin_amdgcn_readfirstlane(at);
#pragma unroll
                for (int u = 0; u < kPairFlight; ++u)
                    if (got[u]) found[mine++] = nb[u];
            }
            BC_FULL_EXEC();
            if (__ballot(a.e < a.re) == 0ull) break;
            next_arcs(d.g, a);
        }
        if (v >= 0) {
            if (L == 0) acc = 1.0;
            if (kExt) {
                if (acc >= 0x1p512) {
                    const int k = ilogb(acc);
                    acc = ldexp(acc, -k);
                    E += k;
                }
                ex[v] = E;
            } else if (!(acc <= kPairRange)) {
                *d.range = 1;
            }
            val[v] = acc;
            q[sg.start + i] = (int32_t)((uint32_t)v | mask << kMaskShift);
            ++wk.owners;
        }
        __syncthreads();
        const int32_t total = nfound;
        if (total > 0) {
            if (t == 0) place = atomicAdd(&d.cnt[(size_t)(L + 1) * d.k + s], total);
            __syncthreads();
            const int32_t to = sg.start + sg.count + place;
            for (int32_t j = t; j < total; j += kBlock) q[to + j] = found[j];
        }
        __syncthreads();  // the list is rewritten by the next piece
    }
    if (d.stats) report_pairs(d.stats, 0, wk);
}

// Reverse step of level L >= 1.
template <bool kExt>
__global__ __launch_bounds__(kBlock) void k_pair_reverse(PairDev d, int32_t L, int32_t per) {
    const int32_t s = (int32_t)(blockIdx.x % (uint32_t)turns(d.k));
    const int32_t piece = (int32_t)(blockIdx.x / (uint32_t)turns(d.k));
    if (s >= d.k || L > d.depth[s]) return;
    const Segment sg = segment(d, L, s);
    const bool leaf = L == d.depth[s];
    const int child = (L + 1) % 3;
    const int32_t *q = d.q + (size_t)s * d.stride;
    const uint8_t *code = d.code + (size_t)s * d.stride;
    double *val = d.val + (size_t)s * d.stride;
    const int32_t *ex = kExt ? d.ex + (size_t)s * d.stride : nullptr;
    double *dl = d.delta + (size_t)s * d.stride;
    PairWork wk;
    for (int32_t i0 = piece * kBlock; i0 < sg.count; i0 += per * kBlock) {
        const int32_t i = i0 + (int32_t)threadIdx.x;
        int32_t v = -1, ev = 0;
        uint32_t mask = 0;
        double sig = 1.0;
        if (i < sg.count) {
            const int32_t x = q[sg.start + i];
            v = entry_vertex(x);
            mask = entry_mask(x);
            sig = val[v];
            if (kExt) ev = ex[v];
        }
        Arcs a = first_arcs(d.g, v, four_of(d.g, leaf ? -1 : v));
        double acc = 0.0;
        for (bool first = true;; first = false) {
            const int32_t (&nb)[4] = a.nb;
            bool down[kPairFlight];
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u)
                down[u] = nb[u] >= 0 && (first ? (mask >> u) & 1u : code[nb[u]] == child);
            double x[kPairFlight];
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u) {
                x[u] = 0.0;
                if (down[u]) {
                    x[u] = val[nb[u]];
                    // c_w sigma_v = (c~_w sigma~_v) 2^(e_v - e_w)
                    if (kExt) x[u] = scaled(x[u], ev - ex[nb[u]]);
                }
            }
#pragma unroll
            for (int u = 0; u < kPairFlight; ++u) {
                acc += x[u];
                wk.arcs += nb[u] >= 0 ? 1u : 0u;
                wk.hits += down[u] ? 1u : 0u;
            }
            BC_FULL_EXEC();
            if (__ballot(a.e < a.re) == 0ull) break;
            next_arcs(d.g, a);
        }
        if (v >= 0) {
            const double delta = sig * acc;
            val[v] = (1.0 + delta) / sig;
            dl[v] = delta;
            ++wk.owners;
        }
    }
    if (d.stats) report_pairs(d.stats, 6, wk);
}

// ---- one workgroup per source -------------------------------------------------

// Where levels are narrow, a level step above is mostly its launch and the
// waits of one short chain.  Here a workgroup runs a whole source, levels
// divided by workgroup barriers, with a visited bit per vertex in LDS, the
// queue's counter in LDS, and the values in global memory by the sign rule of
// bc_source.hip: 0 until a vertex's level, then +value on even levels and
// -value on odd ones, so a sum over the arcs takes max(+-value, 0) of every
// neighbour and needs no level array.  delta[v] takes the place of the forward
// value once the reverse pass has read sigma from the queue-ordered copy.
constexpr int kDeepBlock = 1024;

template <bool kExt>
__global__ __launch_bounds__(kDeepBlock) void k_deep_forward(PairDev d) {
    extern __shared__ uint32_t seen[];  // (n + 31) / 32 words
    __shared__ int32_t cnt[3];          // level L+1's vertices in cnt[(L + 1) % 3]
    const int32_t s = blockIdx.x;
    const int t = threadIdx.x;
    const int32_t words = (d.n + 31) / 32;
    int32_t *q = d.q + (size_t)s * d.stride;
    double *sig = d.sig + (size_t)s * d.stride;
    double *val = d.delta + (size_t)s * d.stride;
    int32_t *ex = kExt ? d.ex + (size_t)s * d.stride : nullptr;
    int32_t *lvl = d.lvl + (size_t)s * d.lcap;
    const int32_t src = d.pos[d.src[s]];
    for (int32_t w = t; w < words; w += kDeepBlock) seen[w] = w == src >> 5 ? 1u << (src & 31) : 0u;
    if (t < 3) cnt[t] = 0;
    if (t == 0) {
        q[0] = src;
        d.at[s] = src;
    }
    __syncthreads();
    PairWork wk;
    int32_t lo = 0, hi = 1, L = 0;
    for (;;) {
        if (t == 0) {
            cnt[(L + 2) % 3] = 0;
            lvl[L] = lo;
        }
        int32_t *next = &cnt[(L + 1) % 3];
        const double par = (L & 1) ? 1.0 : -1.0;  // sign of level L-1
        // (a piece's vertices are loaded two pieces ahead and their arcs one)
        int32_t v0 = lo + t < hi ? q[lo + t] : -1;
        int32_t v1 = lo + t + kDeepBlock < hi ? q[lo + t + kDeepBlock] : -1;
        int4 f0 = four_of(d.g, v0);
        for (int32_t i = lo + t; i - t < hi; i += kDeepBlock) {
            const int32_t v = v0;
            const int4 f = f0;
            f0 = four_of(d.g, v1);
            v0 = v1;
            v1 = i + 2 * kDeepBlock < hi ? q[i + 2 * kDeepBlock] : -1;
            Arcs a = first_arcs(d.g, v, f);
            double acc = 0.0;
            int32_t E = 0;
            uint32_t mask = 0;
            for (bool first = true;; first = false) {
                bool old[4], got[4];
                double x[4];
                int32_t xe[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    old[u] = a.nb[u] >= 0 && ((seen[a.nb[u] >> 5] >> (a.nb[u] & 31)) & 1u);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double y = old[u] ? val[a.nb[u]] : 0.0;
                    // (a value yet to come: claimed for the next level, or at
                    // this level and not done yet, which adds 0 later)
                    if (first && a.nb[u] >= 0 && y == 0.0) mask |= 1u << u;
                    x[u] = fmax(par * y, 0.0);
                    xe[u] = kExt && old[u] ? ex[a.nb[u]] : 0;
                    got[u] = false;
                    if (a.nb[u] >= 0 && !old[u]) {
                        const uint32_t bit = 1u << (a.nb[u] & 31);
                        got[u] = (atomicOr(&seen[a.nb[u] >> 5], bit) & bit) == 0u;
                    }
                }
                BC_FULL_EXEC();
                uint64_t m[4], any = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    m[u] = __ballot(got[u]);
                    any |= m[u];
                    if (kExt) {
                        if (x[u] > 0.0) {
                            if (acc == 0.0) E = xe[u];
                            const int32_t top = E > xe[u] ? E : xe[u];
                            acc = scaled(acc, E - top) + scaled(x[u], xe[u] - top);
                            E = top;
                        }
                    } else {
                        acc += x[u];
                    }
                    wk.arcs += a.nb[u] >= 0 ? 1u : 0u;
                    wk.hits += x[u] > 0.0 ? 1u : 0u;
                }
                if (any) {
                    int32_t all = 0, mine = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        all += (int32_t)__popcll(m[u]);
                        mine = (int32_t)__builtin_amdgcn_mbcnt_hi(
                            (uint32_t)(m[u] >> 32),
                            __builtin_amdgcn_mbcnt_lo((uint32_t)m[u], (uint32_t)mine));
                    }
                    int32_t at = 0;
                    if (lane_id() == 0) at = atomicAdd(next, all);
                    mine += hi + __builtin_amdgcn_readfirstlane(at);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (got[u]) q[mine++] = a.nb[u];
                }
                BC_FULL_EXEC();
                if (__ballot(a.e < a.re) == 0ull) break;
                next_arcs(d.g, a);
            }
            if (v >= 0) {
                if (L == 0) acc = 1.0;
                if (kExt) {
                    if (acc >= 0x1p512) {
                        const int k = ilogb(acc);
                        acc = ldexp(acc, -k);
                        E += k;
                    }
                    ex[v] = E;
                } else if (!(acc <= kPairRange)) {
                    *d.range = 1;
                }
                val[v] = -par * acc;
                sig[i] = acc;
                q[i] = (int32_t)((uint32_t)v | mask << kMaskShift);
                ++wk.owners;
            }
        }
        __syncthreads();
        const int32_t k = *next;
        if (k == 0 || L + 2 >= d.lcap) {
            if (t == 0) {
                lvl[L + 1] = hi;
                // (levels left over: the host runs the source with more room)
                d.depth[s] = k == 0 ? L : -1;
            }
            break;
        }
        lo = hi;
        hi += k;
        ++L;
    }
    if (d.stats) report_pairs(d.stats, 0, wk);
}

template <bool kExt>
__global__ __launch_bounds__(kDeepBlock) void k_deep_reverse(PairDev d) {
    const int32_t s = blockIdx.x;
    const int t = threadIdx.x;
    const int32_t *q = d.q + (size_t)s * d.stride;
    const double *sig = d.sig + (size_t)s * d.stride;
    double *c = d.val + (size_t)s * d.stride;
    double *delta = d.delta + (size_t)s * d.stride;
    const int32_t *ex = kExt ? d.ex + (size_t)s * d.stride : nullptr;
    const int32_t *lvl = d.lvl + (size_t)s * d.lcap;
    const int32_t deepest = d.depth[s];
    if (t == 0) delta[entry_vertex(q[0])] = 0.0;  // the source has none
    PairWork wk;
    // The whole queue is known here, so a piece's entries are loaded two
    // pieces ahead and its arcs one, across levels too: a level waits for its
    // children's values and little else.
    struct Piece {
        int32_t L, lo, hi, i0;  // level, its queue positions, the piece's first
    };
    auto start = [&](int32_t L) {
        Piece p{L, 0, 0, 0};
        if (L >= 1) {
            p.lo = lvl[L];
            p.hi = lvl[L + 1];
            p.i0 = p.lo;
        }
        return p;
    };
    auto after = [&](const Piece &p) {
        Piece n = p;
        n.i0 += kDeepBlock;
        return n.i0 < n.hi ? n : start(p.L - 1);
    };
    auto entry = [&](const Piece &p) { return p.i0 + t < p.hi ? q[p.i0 + t] : -1; };
    auto arcs = [&](const Piece &p, int32_t x) {
        return four_of(d.g, x == -1 || p.L == deepest ? -1 : entry_vertex(x));
    };
    Piece p0 = start(deepest), p1 = after(p0);
    int32_t x0 = entry(p0), x1 = entry(p1);
    int4 f0 = arcs(p0, x0);
    while (p0.L >= 1) {
        const Piece p2 = p1.L >= 1 ? after(p1) : p1;
        const int32_t x2 = entry(p2);
        const int4 f1 = arcs(p1, x1);
        const double child = (p0.L & 1) ? 1.0 : -1.0;  // sign of level L+1
        const int32_t v = x0 == -1 ? -1 : entry_vertex(x0);
        const uint32_t mask = x0 == -1 ? 0u : entry_mask(x0);
        const double sg = v >= 0 ? sig[p0.i0 + t] : 1.0;
        const int32_t ev = kExt && v >= 0 ? ex[v] : 0;
        Arcs a = first_arcs(d.g, v, f0);
        double acc = 0.0;
        for (bool first = true;; first = false) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool look = a.nb[u] >= 0 && (!first || ((mask >> u) & 1u));
                x[u] = look ? fmax(child * c[a.nb[u]], 0.0) : 0.0;
                if (kExt && x[u] > 0.0) x[u] = scaled(x[u], ev - ex[a.nb[u]]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc += x[u];
                wk.arcs += a.nb[u] >= 0 ? 1u : 0u;
                wk.hits += x[u] > 0.0 ? 1u : 0u;
            }
            BC_FULL_EXEC();
            if (__ballot(a.e < a.re) == 0ull) break;
            next_arcs(d.g, a);
        }
        if (v >= 0) {
            const double dl = sg * acc;
            c[v] = -child * ((1.0 + dl) / sg);
            delta[v] = dl;
            ++wk.owners;
        }
        if (p1.L != p0.L) __syncthreads();  // the level is done
        p0 = p1;
        p1 = p2;
        x0 = x1;
        x1 = x2;
        f0 = f1;
    }
    if (d.stats) report_pairs(d.stats, 6, wk);
}

// The two value arrays cleared (a vertex that a source does not reach has no
// dependency, and adds nothing to a sum).
__global__ void k_deep_clear(PairDev d) {
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    double2 *a = reinterpret_cast<double2 *>(d.val), *b = reinterpret_cast<double2 *>(d.delta);
    for (size_t i = tid; i < (size_t)d.k * d.stride / 2; i += step) {
        a[i] = make_double2(0.0, 0.0);
        b[i] = make_double2(0.0, 0.0);
    }
    if (tid == 0) *d.range = 0;
}

// code = 3 everywhere, the counters cleared.
__global__ void k_pair_clear(PairDev d) {
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    const uint4 unreached = make_uint4(0x03030303u, 0x03030303u, 0x03030303u, 0x03030303u);
    for (size_t i = tid; i < (size_t)d.k * d.stride / 16; i += step)
        reinterpret_cast<uint4 *>(d.code)[i] = unreached;
    for (size_t i = tid; i < (size_t)d.k * d.lcap; i += step) d.cnt[i] = 0;
    if (tid == 0) *d.range = 0;
}

__global__ void k_pair_seed(PairDev d) {
    const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= d.k) return;
    const int32_t v = d.pos[d.src[s]];
    d.at[s] = v;
    d.q[(size_t)s * d.stride] = v;
    d.code[(size_t)s * d.stride + v] = 0;
    d.cnt[s] = 1;
    d.lvl[s] = 0;
    d.depth[s] = 0;
}

// out[caller id] (+)= the sources' dependencies on each vertex: kPairSum at a
// time by a tree, the groups added in order (a later round's to the earlier
// rounds' sum one by one, as if they were one round's).
__global__ __launch_bounds__(kBlock) void k_pair_sum(PairDev d, const int32_t *caller, double *out,
                                                     int32_t carry) {
    const int32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v >= d.n) return;
    const int32_t o = caller[v];
    double sum = carry ? out[o] : 0.0;
    for (int32_t s0 = 0; s0 < d.k; s0 += kPairSum) {
        int c[kPairSum];
        double x[kPairSum];
#pragma unroll
        for (int j = 0; j < kPairSum; ++j) {
            c[j] = s0 + j < d.k ? (d.code ? d.code[(size_t)(s0 + j) * d.stride + v] : 0) : 3;
            x[j] = 0.0;
            // (with codes, the source itself has no dependency written)
            if (c[j] != 3 && !(d.code && d.at[s0 + j] == v))
                x[j] = d.delta[(size_t)(s0 + j) * d.stride + v];
        }
#pragma unroll
        for (int w = kPairSum / 2; w >= 1; w /= 2)
#pragma unroll
            for (int j = 0; j < w; ++j) x[j] += x[j + w];
        sum += x[0];
    }
    out[o] = sum;
}

}  // namespace

#ifdef BC_CHECK_EXEC
unsigned int exec_partial_pair() { return exec_partial_take(); }
#endif

hipError_t pair_start(const PairDev &d, hipStream_t stream) {
    const size_t pieces = (size_t)d.k * d.stride / 16 / kBlock;
    const int grid = (int)(pieces < 1 ? 1 : (pieces > 4096 ? 4096 : pieces));
    hipLaunchKernelGGL(k_pair_clear, dim3(grid), dim3(kBlock), 0, stream, d);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pair_seed, dim3((d.k + kBlock - 1) / kBlock), dim3(kBlock), 0, stream, d);
    return hipGetLastError();
}

hipError_t pair_forward(const PairDev &d, int32_t level, int32_t per, hipStream_t stream) {
    hipLaunchKernelGGL(d.ex ? k_pair_forward<true> : k_pair_forward<false>, dim3(turns(d.k) * per),
                       dim3(kBlock), 0, stream, d, level, per);
    return hipGetLastError();
}

hipError_t pair_reverse(const PairDev &d, int32_t level, int32_t per, hipStream_t stream) {
    hipLaunchKernelGGL(d.ex ? k_pair_reverse<true> : k_pair_reverse<false>, dim3(turns(d.k) * per),
                       dim3(kBlock), 0, stream, d, level, per);
    return hipGetLastError();
}

hipError_t deep_source(const PairDev &d, int pass, hipStream_t stream) {
    if (pass == 0) {
        const size_t pieces = (size_t)d.k * d.stride / 2 / kBlock;
        const int grid = (int)(pieces < 1 ? 1 : (pieces > 8192 ? 8192 : pieces));
        hipLaunchKernelGGL(k_deep_clear, dim3(grid), dim3(kBlock), 0, stream, d);
    } else if (pass == 1) {
        hipLaunchKernelGGL(d.ex ? k_deep_forward<true> : k_deep_forward<false>, dim3(d.k),
                           dim3(kDeepBlock), deep_lds_bytes(d.n), stream, d);
    } else {
        hipLaunchKernelGGL(d.ex ? k_deep_reverse<true> : k_deep_reverse<false>, dim3(d.k),
                           dim3(kDeepBlock), 0, stream, d);
    }
    return hipGetLastError();
}

size_t deep_lds_bytes(int32_t n) { return ((size_t)n + 31) / 32 * sizeof(uint32_t); }

hipError_t pair_sum(const PairDev &d, const int32_t *caller, double *out, bool carry,
                    hipStream_t stream) {
    hipLaunchKernelGGL(k_pair_sum, dim3((d.n + kBlock - 1) / kBlock), dim3(kBlock), 0, stream, d,
                       caller, out, carry ? 1 : 0);
    return hipGetLastError();
}

}  // namespace bcx
