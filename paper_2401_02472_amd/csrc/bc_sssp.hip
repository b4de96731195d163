// Single-source shortest paths over weighted arcs: the paper's fixed-point
// formulation (Sections "fixedPoint Construct" and "Min/Max Constructs").  A
// pass relaxes the out-arcs of every vertex modified in the previous pass,
// <nbr.dist, nbr.modified> = <Min(nbr.dist, v.dist + w), true>, with an atomic
// min on the distance; the passes repeat until one modifies nothing.
//
// Instead of two modified arrays that must be cleared, a vertex carries the
// number of the pass that must process it (stamp): a pass p takes the
// vertices stamped p and stamps p + 1 on the ones it improves.  (The distance
// of its last turn in place of the stamp saves the second write of an
// improvement, but vertices then take their turn in the pass that improves
// them, at distances that are not final yet: 0.49 -> 0.69 ms on the
// 262K-vertex R-MAT.)  A pass that has much to do takes only the vertices
// within delta of the smallest pending distance and stamps the others p + 1,
// so that fewer vertices relax their arcs again; one with little to do takes
// all.  Each pass leaves its successor an estimate of the pending arcs and the
// smallest pending distance.
//
// Passes are launched over the same work items as the batched BC kernels:
// chunk items of 512 arcs for vertices of degree > 64, and 64-vertex groups
// whose arcs are flattened into runs of 64 (one arc per lane).  Distances are
// exact integers, so the result does not depend on the order of the
// relaxations.
#include "bc_internal.h"
#include "bc_wave.h"

namespace bcx {
namespace {

constexpr int kPerLane = kChunk / kWave;  // arcs per lane in a chunk item
static_assert(kPerLane * kWave == kChunk, "a chunk item is kPerLane arcs per lane");

constexpr int32_t kInf = 0x7fffffff;
static_assert(kSsspSlots == kWave, "a wave reads a pass's slots at once");

// Vertices with a copy of their distance in LDS (4 KB: scale-22 R-MAT 2.10 ms
// and 2M-vertex uniform graph 1.52; 16 KB 2.15 and 1.66; with 159 KB in one
// workgroup per CU 1.94 and 1.66, but scale 18 0.50 in place of 0.44).
constexpr int32_t kHubs = 1024;
constexpr int kGroups = 4;        // groups of 64 vertices whose stamps load together
constexpr int kRuns = 4;          // runs of 64 flattened arcs in flight

struct Relax {
    uint32_t active = 0, arcs = 0, better = 0;  // work counters (per lane)
    uint32_t work = 0;                          // arcs left to the next pass, about
    uint32_t key = 0;                           // kInf - the smallest distance left to it
    __device__ __forceinline__ void leave(uint32_t arcs_left, int32_t dist) {
        work += arcs_left;
        key = max(key, (uint32_t)(kInf - dist));
    }
};

// About the arcs of v (ids are degree-descending; the prefixes are the
// vertices of degree > 512, > 64 and > 8).
__device__ __forceinline__ uint32_t about_arcs(const SsspDev &d, int32_t v) {
    return v >= d.big_end ? (v < d.mid_end ? 24 : 4) : (v < d.multi_end ? 1500 : 200);
}

// Relax kArcs arcs per lane to the vertices nb[] (-1: none) at distances nd[].
// The first `hubs` vertices have a copy of their distance in LDS, which takes
// the minimum first: a hub that thousands of vertices improve at once sees
// one atomic from a workgroup for each new minimum there (346 -> 26 us for the
// pass that reaches the hubs of the scale-22 R-MAT).  Loads and atomics of
// kTogether arcs are issued together.
template <bool kWait, int kTogether, int kArcs>
__device__ __forceinline__ void relax(const SsspDev &d, int32_t *hub, int32_t hubs,
                                      const int32_t (&nb)[kArcs], const int32_t (&nd)[kArcs],
                                      int32_t pass, Relax &r) {
    int32_t old[kArcs];
#pragma unroll
    for (int at = 0; at < kArcs; at += kTogether) {
#pragma unroll
        for (int u = at; u < at + kTogether; ++u) {
            old[u] = -1;
            if (nb[u] >= hubs) old[u] = d.dist[nb[u]];
            else if (nb[u] >= 0 && nd[u] < hub[nb[u]]) old[u] = atomicMin(&hub[nb[u]], nd[u]);
        }
        // kWait: wait for the distance found, so that only the improvements are
        // stamped (there are more tries than those on graphs with hubs).  Without
        // it every try is stamped, which is right too: a distance above nd was
        // read, so someone improved the vertex in this pass (the 1M-vertex grid
        // 1.67 -> 1.45 ms; the scale-22 R-MAT the other way 2.10 -> 2.15).
#pragma unroll
        for (int u = at; u < at + kTogether; ++u) {
            if (nd[u] < old[u]) {
                if (kWait || d.stats) old[u] = atomicMin(&d.dist[nb[u]], nd[u]);
                else atomicMin(&d.dist[nb[u]], nd[u]);
            }
        }
#pragma unroll
        for (int u = at; u < at + kTogether; ++u) {
            if (nd[u] < old[u]) {
                d.stamp[nb[u]] = pass + 1;
                r.leave(about_arcs(d, nb[u]), nd[u]);
                ++r.better;
            }
        }
    }
}

__device__ __forceinline__ int32_t weight_of(const SsspDev &d, int32_t e) {
    return d.weight ? d.weight[e] : 1;
}

// One pass.  left: three sets of slots, of which pass p reads the one of pass
// p - 1, adds to its own and clears the one of pass p + 1.  A pass that finds
// nothing pending returns at once, so that several passes can be queued without
// a host wait.  *chose is set by a pass that leaves vertices to later ones.
//
// A wave looks at 64 chunk items at once, one per lane, and then relaxes the
// pending ones with all 64 lanes, the next item's columns and weights loading
// during the distance reads (one item after the other, each waiting for its
// table row and stamp, took 75 us on the scale-22 R-MAT with nothing pending).
//
// On the scale-22 R-MAT (source of the measured workload) 17 passes take 1.8 ms
// of 2.06, 1.3 of them the three that relax 100M arcs: the 12M improvements,
// each a 4-byte atomic and a 4-byte store at random, bound those.  Before, with
// every pass taking all: 11 passes, 3 times every arc, 42M improvements, 2.4 ms.
// The waves per SIMD asked for: 1M-vertex grid 1.43 ms with 8, 1.56 with 6.
//
// Three forms: kSplit, where a pass may choose; without it, and kWait, large
// graphs of even weights, which relax one arc after the other, as a level's
// arcs all offer the same distance and later ones find it there (scale-16
// R-MAT 0.21 -> 0.17 ms, scale 20 0.37, where kSplit takes 0.55); and
// neither, small graphs and narrow fronts.
template <bool kSplit, bool kWait>
__global__ __launch_bounds__(kBlock, kSplit ? 6 : 8) void k_sssp_pass(SsspDev d, int32_t pass,
                                                                      SsspSlot *left,
                                                                      int32_t *chose) {
    __shared__ int32_t hub[kSplit ? kHubs : 1];
    constexpr bool kSerial = kWait && !kSplit;
    const int lane = lane_id();
    const SsspSlot *prev = left + (pass + 2) % 3 * kSsspSlots;
    SsspSlot *cur = left + pass % 3 * kSsspSlots;
    if (blockIdx.x == 0 && threadIdx.x < kSsspSlots)
        left[(pass + 1) % 3 * kSsspSlots + threadIdx.x] = SsspSlot{};
    unsigned long long due = kSplit ? prev[lane].work : prev[0].work;
    uint32_t key = kSplit ? prev[lane].key : 0;
    if constexpr (kSplit) {
        BC_FULL_EXEC();
#pragma unroll
        for (int off = kSsspSlots / 2; off >= 1; off >>= 1) {
            due += __shfl_xor(due, off);
            key = max(key, __shfl_xor(key, off));
        }
        due = shfl64(due, 0);
        key = __shfl(key, 0);
    }
    if (due == 0) return;
    const bool split = kSplit && (int64_t)due > d.split;
    if (split && blockIdx.x == 0 && threadIdx.x == 0) *chose = 1;
    const int64_t cut = split ? (int64_t)kInf - key + d.delta : kInf;
    const int32_t limit = (int32_t)min(cut, (int64_t)kInf);  // distances below it are taken
    int32_t hubs = 0;
    if constexpr (kSplit) {
        hubs = min(d.n, kHubs);
        for (int32_t i = threadIdx.x; i < hubs; i += kBlock) hub[i] = d.dist[i];
        __syncthreads();
    }
    constexpr int kWaves = kWavesPerBlock;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + threadIdx.x / kWave);
    const uint32_t nwaves = gridDim.x * kWaves;
    Relax r;
    for (uint32_t first = wave; first < d.items; first += kWave * nwaves) {
        const uint32_t it = first + (uint32_t)lane * nwaves;
        int32_t v = -1, cb = 0, ce = 0, dv = 0;
        bool mine = false;
        if (it < d.items) {
            const int2 info = d.item_info[it];
            v = info.x;
            if (d.stamp[v] == pass) {
                dv = d.dist[v];
                cb = d.row_ptr[v] + info.y * kChunk;
                ce = min(d.row_ptr[v + 1], cb + kChunk);
                mine = dv < limit;
                if (!mine) {
                    d.stamp[v] = pass + 1;
                    r.leave((uint32_t)(ce - cb) + 1, dv);
                } else if (info.y == 0) {
                    ++r.active;
                }
            }
        }
        uint64_t todo = __ballot(mine);
        int32_t c[kPerLane], w[kPerLane];
        auto arcs = [&](int i, int32_t(&col)[kPerLane], int32_t(&wt)[kPerLane]) {
            const int32_t b = __builtin_amdgcn_readlane(cb, i);
            const int32_t e = __builtin_amdgcn_readlane(ce, i);
#pragma unroll
            for (int u = 0; u < kPerLane; ++u) {
                col[u] = -1;
                wt[u] = 0;
                if (b + u * kWave < e) {
                    const int32_t a = b + u * kWave + lane;
                    if (a < e) {
                        col[u] = d.col_idx[a];
                        wt[u] = weight_of(d, a);
                    }
                }
            }
        };
        if (todo) arcs(__builtin_ctzll(todo), c, w);
        while (todo) {
            const int i = __builtin_ctzll(todo);
            todo &= todo - 1;
            int32_t c2[kPerLane], w2[kPerLane];
            arcs(todo ? __builtin_ctzll(todo) : i, c2, w2);
            const int32_t from = __builtin_amdgcn_readlane(dv, i);
#pragma unroll
            for (int u = 0; u < kPerLane; ++u) {
                r.arcs += c[u] >= 0 ? 1u : 0u;
                // (saturated: the farthest vertex's arcs may pass the range)
                w[u] = (int32_t)min((uint32_t)from + (uint32_t)w[u], (uint32_t)kInf);
            }
            relax<kWait, kSerial ? 1 : kPerLane>(d, hub, hubs, c, w, pass, r);
#pragma unroll
            for (int u = 0; u < kPerLane; ++u) {
                c[u] = c2[u];
                w[u] = w2[u];
            }
        }
    }
    // 64 vertices of degree 1 to 64: the arcs of the pending ones, flattened.
    // The stamps of the wave's next kGroups groups load together.
    const uint32_t groups = (uint32_t)((d.live_end - d.big_end + kWave - 1) / kWave);
    // (dealt on from where the items end, so that few waves get both)
    const uint32_t after = d.items % nwaves;
    const uint32_t gwave = wave >= after ? wave - after : wave + nwaves - after;
    for (uint32_t g0 = gwave; g0 < groups; g0 += kGroups * nwaves) {
        uint32_t mine = 0;  // bit q: the lane's vertex of group q is pending
#pragma unroll
        for (int q = 0; q < kGroups; ++q) {
            const int64_t v = d.big_end + ((int64_t)g0 + (int64_t)q * nwaves) * kWave + lane;
            const int32_t st = v < d.live_end ? d.stamp[v] : 0;
            mine |= st == pass ? 1u << q : 0u;
        }
#pragma unroll 1
        for (int q = 0; q < kGroups; ++q) {
            const bool pending = (mine >> q & 1) != 0;
            if (__ballot(pending) == 0) continue;
            const int32_t me = d.big_end + (int32_t)(g0 + q * nwaves) * kWave + lane;
            int32_t rs = 0, cnt = 0, dv = 0;
            if (pending) {
                dv = d.dist[me];
                rs = d.row_ptr[me];
                cnt = d.row_ptr[me + 1] - rs;
                if (dv < limit) {
                    ++r.active;
                } else {
                    d.stamp[me] = pass + 1;
                    r.leave((uint32_t)cnt + 1, dv);
                    cnt = 0;
                }
            }
            if (__ballot(cnt > 0) == 0) continue;
            uint32_t total;
            const uint32_t excl = wave_excl_scan((uint32_t)cnt, total);
            for (uint32_t c0 = 0; c0 < total; c0 += kRuns * kWave) {
                int32_t c[kRuns], w[kRuns];
#pragma unroll
                for (int u = 0; u < kRuns; ++u) {
                    c[u] = -1;
                    w[u] = 0;
                    if (c0 + u * kWave < total) {
                        const uint32_t a = c0 + u * kWave + (uint32_t)lane;
                        const int o = owner_lane(excl, a);
                        const int32_t o_rs = __shfl(rs, o);
                        const uint32_t o_excl = __shfl(excl, o);
                        const int32_t o_dv = __shfl(dv, o);
                        if (a < total) {
                            const int32_t e = o_rs + (int32_t)(a - o_excl);
                            c[u] = d.col_idx[e];
                            w[u] = (int32_t)min((uint32_t)o_dv + (uint32_t)weight_of(d, e),
                                                (uint32_t)kInf);
                            ++r.arcs;
                        }
                    }
                }
                relax<kWait, kSerial ? 1 : kRuns>(d, hub, hubs, c, w, pass, r);
            }
        }
    }
    if constexpr (!kSplit) {
        BC_FULL_EXEC();
        if (__ballot(r.work != 0) && lane == 0) cur->work = 1;
    } else {
        // what is left, per workgroup
        __shared__ uint32_t s_work[kWaves], s_key[kWaves];
        BC_FULL_EXEC();
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            r.work += __shfl_xor(r.work, off);
            r.key = max(r.key, __shfl_xor(r.key, off));
        }
        if (lane == 0) {
            s_work[threadIdx.x / kWave] = r.work;
            s_key[threadIdx.x / kWave] = r.key;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long work = 0;
            uint32_t best = 0;
            for (int w = 0; w < kWaves; ++w) {
                work += s_work[w];
                best = max(best, s_key[w]);
            }
            if (work > 0) {
                SsspSlot *mine = cur + blockIdx.x % kSsspSlots;
                atomicAdd(&mine->work, work);
                atomicMax(&mine->key, best);
            }
        }
    }
    if (d.stats) {  // one atomic per workgroup and counter: they share a line
        __shared__ unsigned long long s_stats[3];
        if (threadIdx.x < 3) s_stats[threadIdx.x] = 0;
        __syncthreads();
        unsigned long long a = r.active, b = r.arcs, c = r.better;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            a += __shfl_xor(a, off);
            b += __shfl_xor(b, off);
            c += __shfl_xor(c, off);
        }
        if (lane == 0 && (a | b | c)) {
            atomicAdd(&s_stats[0], a);
            atomicAdd(&s_stats[1], b);
            atomicAdd(&s_stats[2], c);
        }
        __syncthreads();
        if (threadIdx.x < 3 && s_stats[threadIdx.x])
            atomicAdd(&d.stats[threadIdx.x], s_stats[threadIdx.x]);
    }
}

// What the passes so far left to the next one, in slot 0 alone (a pass without
// kSplit looks at no other), and for the host: flags[0] = something is pending.
__global__ __launch_bounds__(kSsspSlots) void k_sssp_fold(SsspSlot *set, int32_t *flags) {
    unsigned long long work = set[threadIdx.x].work;
    uint32_t key = set[threadIdx.x].key;
#pragma unroll
    for (int off = kSsspSlots / 2; off >= 1; off >>= 1) {
        work += __shfl_xor(work, off);
        key = max(key, __shfl_xor(key, off));
    }
    const bool first = threadIdx.x == 0;
    set[threadIdx.x] = SsspSlot{first ? work : 0, first ? key : 0, {}};
    if (first) flags[0] = work != 0 ? 1 : 0;
}

// Distances and stamps for pass 1; its predecessor's slots say "one arc, at 0".
__global__ void k_sssp_init(SsspDev d, int32_t src, SsspSlot *left, int32_t *flags) {
    const int32_t at = blockIdx.x * blockDim.x + threadIdx.x, all = gridDim.x * blockDim.x;
    if (at < 2) flags[at] = 0;
    for (int32_t i = at; i < 3 * kSsspSlots; i += all)
        left[i] = SsspSlot{i == 0, i == 0 ? (uint32_t)kInf : 0, {}};
    for (int32_t v = at; v < d.n; v += all) {
        d.dist[v] = v == src ? 0 : kInf;
        d.stamp[v] = v == src ? 1 : 0;
    }
}

// dist in caller order, -1 where unreachable.
__global__ void k_sssp_export(int32_t n, const int32_t *perm, const int32_t *dist,
                              int32_t *out) {
    for (int32_t o = blockIdx.x * blockDim.x + threadIdx.x; o < n; o += gridDim.x * blockDim.x) {
        const int32_t x = dist[perm[o]];
        out[o] = x == kInf ? -1 : x;
    }
}

// new_vals[e] = old_vals[e'] where e' is the same arc in the caller's CSR
// (rows are permuted, the arcs of a row keep their order).
__global__ void k_permute_arcs(int32_t n, int64_t nnz, const int32_t *old_rp,
                               const int32_t *old_vals, const int32_t *new_rp,
                               const int32_t *iperm, int32_t *new_vals) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += stride) {
        int32_t lo = 0, hi = n - 1;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo + 1) / 2;
            if ((int64_t)new_rp[mid] <= e) lo = mid;
            else hi = mid - 1;
        }
        new_vals[e] = old_vals[(int64_t)old_rp[iperm[lo]] + (e - new_rp[lo])];
    }
}

int blocks_for(int64_t n) {
    int64_t b = (n + kBlock - 1) / kBlock;
    return (int)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

}  // namespace

#ifdef BC_CHECK_EXEC
unsigned int exec_partial_sssp() { return exec_partial_take(); }
#endif

hipError_t sssp_init(const SsspDev &d, int32_t src, SsspSlot *left, int32_t *flags,
                     hipStream_t stream) {
    hipLaunchKernelGGL(k_sssp_init, dim3(blocks_for(d.n)), dim3(kBlock), 0, stream, d, src, left,
                       flags);
    return hipGetLastError();
}

hipError_t sssp_pass(const SsspDev &d, int32_t pass, SsspSlot *left, int32_t *chose,
                     hipStream_t stream) {
    const int64_t groups = (d.live_end - d.big_end + kWave - 1) / kWave;
    int64_t blocks = (d.items + groups + kWavesPerBlock - 1) / kWavesPerBlock;
    blocks = blocks < 1 ? 1 : (blocks > kMaxGridBlocks ? kMaxGridBlocks : blocks);
    auto k = d.split >= 0 ? k_sssp_pass<true, true>
                          : (d.wait ? k_sssp_pass<false, true> : k_sssp_pass<false, false>);
    hipLaunchKernelGGL(k, dim3((int)blocks), dim3(kBlock), 0, stream, d, pass, left, chose);
    return hipGetLastError();
}

hipError_t sssp_fold(int32_t pass, SsspSlot *left, int32_t *pending, hipStream_t stream) {
    hipLaunchKernelGGL(k_sssp_fold, dim3(1), dim3(kSsspSlots), 0, stream,
                       left + pass % 3 * kSsspSlots, pending);
    return hipGetLastError();
}

hipError_t sssp_export(int32_t n, const int32_t *perm, const int32_t *dist, int32_t *out,
                       hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sssp_export, dim3(blocks_for(n)), dim3(kBlock), 0, stream, n, perm, dist,
                       out);
    return hipGetLastError();
}

hipError_t permute_arc_values(int32_t n, int64_t nnz, const int32_t *old_rp,
                              const int32_t *old_vals, const int32_t *new_rp,
                              const int32_t *iperm, int32_t *new_vals, hipStream_t stream) {
    if (n == 0 || nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(k_permute_arcs, dim3(blocks_for(nnz)), dim3(kBlock), 0, stream, n, nnz,
                       old_rp, old_vals, new_rp, iperm, new_vals);
    return hipGetLastError();
}

}  // namespace bcx
