// PageRank: the paper's pull iteration (the generated loop of Section "Backend
// Optimizations", OpenACC reduction).  Every vertex starts at 1/n; an
// iteration computes sum = sum over the arcs u->v of pr[u] / outdeg(u),
// val = (1 - d)/n + d * sum and the L1 change sum |val - pr[v]|, into a second
// buffer; iterations stop when the change is at most tol or after max_iter.
//
// pr[u] / outdeg(u) is kept per vertex (contrib, written with the rank), so
// an arc costs one 8-byte gather.  Sums run over the reversed CSR in the
// work layout of the batched BC kernels: vertices of degree <= 64 64 at a
// time with 1 to 8 lanes to a vertex, vertices up to 512 arcs one wave each
// (tree sum), larger ones one wave per 512-arc chunk with the chunks' partial
// sums added by a second kernel.  The change is summed per wave into slots
// that a third kernel adds in slot order, so every result repeats bit for bit.
//
// Bound: a gather that misses the first-level cache moves a 128-byte line out
// of the L2 (257 G gathers/s at most), and past the L2 81 G/s at 16 MB of
// shares.  Where few vertices own many arcs, every workgroup keeps the shares
// of the 20,352 highest-degree ones in its LDS: on the scale-22 R-MAT
// (128M arcs, 42 % of them theirs) an iteration's pull takes 0.64 ms in place
// of 0.88, with 22M lines from beyond the L2 at 4.4 TB/s; without that, the
// same kernel 0.84.  Loads of the columns that bypass the caches made the
// graphs whose columns fit the last-level cache slower (scale 20 0.127 ->
// 0.172 ms) and gained nothing on the others.
#include "bc_internal.h"
#include "bc_wave.h"

namespace bcx {
namespace {

constexpr int kPerLane = kChunk / kWave;  // arcs per lane in a chunk item
static_assert(kPerLane * kWave == kChunk, "a chunk item is kPerLane arcs per lane");

constexpr int kDiffBlock = 1024;
constexpr int32_t kHubs = kPrHubs;
constexpr int kHubBlock = 1024;  // one workgroup per CU: its LDS holds the hubs' shares
constexpr int kHubBlocks = 256;

__device__ __forceinline__ bool converged(const PrDev &d, int32_t iter) {
    return iter > 0 && d.diff[iter - 1] >= 0.0 && d.diff[iter - 1] <= d.tol;
}

// New rank of v from its sum: rank, its per-arc share and the change.
__device__ __forceinline__ double settle_rank(const PrDev &d, int32_t v, double sum,
                                              const double *pr, double *pr_next,
                                              double *contrib_next) {
    const double val = d.base + d.damping * sum;
    pr_next[v] = val;
    const int32_t od = d.row_ptr[v + 1] - d.row_ptr[v];
    contrib_next[v] = od > 0 ? val / (double)od : 0.0;
    return fabs(val - pr[v]);
}

__device__ __forceinline__ void report_diff(const PrDev &d, int set, int32_t wave, double x) {
    x = wave_sum(x);
    if (lane_id() == 0) d.slots[(size_t)set * kFrontWaves + wave] = x;
}

// Share of vertex c (-1: an arc that is not there): the kHubs vertices of
// highest degree from LDS, the others from memory.  Exactly one of the two
// terms is not 0.
template <bool kLds>
__device__ __forceinline__ double share(const double *hub, const double *contrib, int32_t c) {
    const int32_t hubs = kLds ? kHubs : 0;
    double x = 0.0;
    if (c >= hubs) x = contrib[c];
    if constexpr (kLds) x += hub[min((uint32_t)c, (uint32_t)kHubs)];
    return x;
}

// Pull step.  A wave takes per_task consecutive chunk items at a time (all
// arcs of a vertex or one chunk of a split one, 8 gathers in flight per lane
// while the next item's columns load; a tree sum per item), or a group of 64
// small vertices.
template <bool kLds, int kThreads>
__global__ __launch_bounds__(kThreads) void k_pr_pull(PrDev d, int32_t iter, int32_t per_task) {
    extern __shared__ double hub[];  // kLds: shares of the first kHubs vertices, then 0
    if (converged(d, iter)) return;
    const double *pr = d.pr[iter & 1];
    const double *contrib = d.contrib[iter & 1];
    double *pr_next = d.pr[(iter + 1) & 1];
    double *contrib_next = d.contrib[(iter + 1) & 1];
    if constexpr (kLds) {
        for (int32_t i = threadIdx.x; i < min(d.n, kHubs); i += kThreads) hub[i] = contrib[i];
        if (threadIdx.x == 0) hub[kHubs] = 0.0;
        __syncthreads();
    }
    constexpr int kWaves = kThreads / kWave;
    const int lane = lane_id();
    const uint32_t groups = (uint32_t)((d.n - d.big_end + kWave - 1) / kWave);
    const uint32_t tasks = (d.items_in + per_task - 1) / per_task;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + threadIdx.x / kWave);
    const uint32_t nwaves = gridDim.x * kWaves;
    double change = 0.0;
    for (uint32_t t = wave; t < tasks + groups; t += nwaves) {
        if (t < tasks) {
            const uint32_t it = t * per_task + lane;
            const int items = (int)min((uint32_t)per_task, d.items_in - t * per_task);
            int32_t v = 0, cb = 0, ce = 0;
            if (lane < items) {
                const int2 info = d.item_info_in[it];
                v = info.x;
                cb = d.row_ptr_in[v] + info.y * kChunk;
                ce = min(d.row_ptr_in[v + 1], cb + kChunk);
            }
            int32_t c[kPerLane], next[kPerLane];
            auto columns = [&](int i, int32_t(&col)[kPerLane]) {
                const int32_t b = __builtin_amdgcn_readlane(cb, i);
                const int32_t e = __builtin_amdgcn_readlane(ce, i);
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) {
                    col[u] = -1;
                    if (b + u * kWave < e) {
                        const int32_t a = b + u * kWave + lane;
                        const int32_t x = d.col_idx_in[min(a, e - 1)];
                        col[u] = a < e ? x : -1;
                    }
                }
            };
            columns(0, c);
            double sum = 0.0;
            for (int i = 0; i < items; ++i) {
                columns(min(i + 1, items - 1), next);
                double x[kPerLane];
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) x[u] = share<kLds>(hub, contrib, c[u]);
                double s = 0.0;
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) s += x[u];
                s = wave_sum(s);
                if (lane == i) sum = s;
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) c[u] = next[u];
            }
            if (lane < items) {
                if (v < d.multi_end) d.partial[it] = sum;
                else change += settle_rank(d, v, sum, pr, pr_next, contrib_next);
            }
        } else {
            // 64 vertices of degree <= 64, degrees falling: 1, 2, 4 or 8 lanes to
            // a vertex, 8 arcs at most to a lane, 64 / lanes vertices at a time
            const int32_t first = d.big_end + (int32_t)(t - tasks) * kWave;
            const int32_t v = first + lane;
            int32_t rs = 0, cnt = 0;
            if (v < d.n) {
                rs = d.row_ptr_in[v];
                cnt = d.row_ptr_in[v + 1] - rs;
            }
            BC_FULL_EXEC();
            int most = cnt;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) most = max(most, __shfl_xor(most, off));
            most = __builtin_amdgcn_readfirstlane(most);
            int lg = 0;  // lanes to a vertex = 1 << lg
            while ((kPerLane << lg) < most) ++lg;
            double sum = 0.0;
            for (int p = 0; p < (1 << lg) && most > 0; ++p) {
                const int who = (p << (6 - lg)) + (lane >> lg);  // this lane's vertex
                const int32_t b = __shfl(rs, who) + (lane & ((1 << lg) - 1));
                const int32_t e = __shfl(rs, who) + __shfl(cnt, who);
                int32_t c[kPerLane];
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) {
                    const int32_t a = b + (u << lg);
                    c[u] = -1;
                    if (a < e) c[u] = d.col_idx_in[a];
                }
                double x[kPerLane];
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) x[u] = share<kLds>(hub, contrib, c[u]);
                double s = 0.0;
#pragma unroll
                for (int u = 0; u < kPerLane; ++u) s += x[u];
                for (int off = (1 << lg) >> 1; off >= 1; off >>= 1) s += __shfl_xor(s, off);
                const double mine = __shfl(s, (lane << lg) & (kWave - 1));
                if ((lane >> (6 - lg)) == p) sum = mine;
            }
            if (v < d.n) change += settle_rank(d, v, sum, pr, pr_next, contrib_next);
        }
    }
    report_diff(d, 0, (int32_t)wave, change);
}

// Split vertices: their chunks' partial sums, 16 lanes to a vertex, then a
// tree sum (one lane's loads in turn took 48 us on the scale-22 R-MAT, where
// this takes 8: the largest vertex has 600 chunks).
constexpr int kFinishLanes = 16;
__global__ __launch_bounds__(kBlock) void k_pr_finish(PrDev d, int32_t iter) {
    if (converged(d, iter)) return;
    const double *pr = d.pr[iter & 1];
    double *pr_next = d.pr[(iter + 1) & 1];
    double *contrib_next = d.contrib[(iter + 1) & 1];
    const int32_t wave = (blockIdx.x * kBlock + threadIdx.x) / kWave;
    const uint32_t j = threadIdx.x % kFinishLanes;
    constexpr int kPerBlock = kBlock / kFinishLanes;
    double change = 0.0;
    for (int32_t v0 = blockIdx.x * kPerBlock; v0 < d.multi_end; v0 += gridDim.x * kPerBlock) {
        const int32_t v = v0 + (int32_t)threadIdx.x / kFinishLanes;
        double s = 0.0;
        if (v < d.multi_end) {
            const uint32_t end = d.item_first_in[v + 1];
#pragma unroll 4
            for (uint32_t i = d.item_first_in[v] + j; i < end; i += kFinishLanes) s += d.partial[i];
        }
        BC_FULL_EXEC();
#pragma unroll
        for (int off = kFinishLanes / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        if (v < d.multi_end && j == 0) change += settle_rank(d, v, s, pr, pr_next, contrib_next);
    }
    report_diff(d, 1, wave, change);
}

// diff[iter] = the slots of both steps added in order (one block).
__global__ __launch_bounds__(kDiffBlock) void k_pr_diff(PrDev d, int32_t iter, int32_t w0,
                                                        int32_t w1) {
    if (converged(d, iter)) return;
    __shared__ double s[kDiffBlock];
    const int t = threadIdx.x;
    double x = 0.0;
    for (int32_t w = t; w < w0; w += kDiffBlock) x += d.slots[w];
    for (int32_t w = t; w < w1; w += kDiffBlock) x += d.slots[(size_t)kFrontWaves + w];
    s[t] = x;
    __syncthreads();
    for (int h = kDiffBlock / 2; h >= 1; h >>= 1) {
        if (t < h) s[t] += s[t + h];
        __syncthreads();
    }
    if (t == 0) d.diff[iter] = s[0];
}

__global__ void k_pr_init(PrDev d, int32_t max_iter) {
    const double r = 1.0 / (double)d.n;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < d.n;
         v += gridDim.x * blockDim.x) {
        d.pr[0][v] = r;
        const int32_t od = d.row_ptr[v + 1] - d.row_ptr[v];
        d.contrib[0][v] = od > 0 ? r / (double)od : 0.0;
    }
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < max_iter;
         i += gridDim.x * blockDim.x)
        d.diff[i] = -1.0;  // iterations not run
}

struct PullShape {
    bool lds;
    int blocks, waves, per_task;  // workgroups, waves of one, chunk items of a task
};

// Hubs in LDS cost a 160 KB load per workgroup and half the waves of a CU:
// they pay from about 8M hub arcs where these are much of the graph (ms per
// iteration, memory only / hubs in LDS: R-MAT scale 22 0.85 / 0.67, 20
// 0.164 / 0.127, 18, with 6M hub arcs, 0.050 / 0.049; uniform random 2M
// vertices 0.435 / 0.442, 500K 0.061 / 0.076; a 1M-vertex grid 0.025 / 0.032).
// Four items to a task read four items' table rows at once, where one item's
// wait for each (scale 16 0.024 / 0.026, 20 0.164 / 0.176); six where every wave has
// several tasks (scale 22 0.66 / 0.68, 20 0.127 / 0.134, but 18 0.063 / 0.049).
PullShape pull_shape(const PrDev &d) {
    PullShape p{};
    p.lds = d.hub_arcs >= (8 << 20) && d.hub_arcs >= d.nnz / 4;
    p.waves = (p.lds ? kHubBlock : kBlock) / kWave;
    const int64_t most = p.lds ? kHubBlocks : kMaxGridBlocks;
    p.per_task = p.lds && d.items_in >= 16 * most * p.waves ? 6 : 4;
    const int64_t tasks = ((int64_t)d.items_in + p.per_task - 1) / p.per_task +
                          ((int64_t)d.n - d.big_end + kWave - 1) / kWave;
    const int64_t b = (tasks + p.waves - 1) / p.waves;
    p.blocks = (int)(b < 1 ? 1 : (b > most ? most : b));
    return p;
}

}  // namespace

#ifdef BC_CHECK_EXEC
unsigned int exec_partial_pagerank() { return exec_partial_take(); }
#endif

hipError_t pagerank_init(const PrDev &d, int32_t max_iter, hipStream_t stream) {
    const int64_t m = d.n > max_iter ? d.n : max_iter;
    int64_t b = (m + kBlock - 1) / kBlock;
    b = b < 1 ? 1 : (b > 4096 ? 4096 : b);
    hipLaunchKernelGGL(k_pr_init, dim3((int)b), dim3(kBlock), 0, stream, d, max_iter);
    return hipGetLastError();
}

hipError_t pagerank_pull(const PrDev &d, int32_t iter, hipStream_t stream) {
    const PullShape p = pull_shape(d);
    if (p.lds)
        hipLaunchKernelGGL((k_pr_pull<true, kHubBlock>), dim3(p.blocks), dim3(kHubBlock),
                           (kHubs + 1) * sizeof(double), stream, d, iter, p.per_task);
    else
        hipLaunchKernelGGL((k_pr_pull<false, kBlock>), dim3(p.blocks), dim3(kBlock), 0, stream, d,
                           iter, p.per_task);
    return hipGetLastError();
}

hipError_t pagerank_finish(const PrDev &d, int32_t iter, hipStream_t stream) {
    const PullShape p = pull_shape(d);
    int g1 = 0;
    if (d.multi_end > 0) {
        const int64_t b = ((int64_t)d.multi_end * kFinishLanes + kBlock - 1) / kBlock;
        g1 = (int)(b < kMaxGridBlocks ? b : kMaxGridBlocks);
        hipLaunchKernelGGL(k_pr_finish, dim3(g1), dim3(kBlock), 0, stream, d, iter);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_pr_diff, dim3(1), dim3(kDiffBlock), 0, stream, d, iter,
                       p.blocks * p.waves, g1 * kWavesPerBlock);
    return hipGetLastError();
}

}  // namespace bcx
