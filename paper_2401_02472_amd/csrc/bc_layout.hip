// A vertex order for the pair path (bc_pair.hip) in which vertices near each
// other in the graph lie near each other in memory.
//
// A level of a road-like graph is a set of rings; with ids in degree order
// (ties in the caller's order) the few ring vertices of a cache line are one
// or two, and the level steps run at the rate of scattered lines.  Here the
// vertices are grown into patches around seed vertices: patches of about 16
// vertices (a cache line of doubles) inside ones of about 128 (a line of
// bytes) inside ones of about 1024, each numbered one after another, so a ring
// meets whole patches.  On the 1024 x 1024 road-like grid with shortcuts, 64
// sources, this and queues that keep the order along the rings take the level
// steps from 24.8 to 15.6 ms.  Which patch a vertex joins, and its place there, only moves data: sums run
// over its arcs in the order of its row, which the copy keeps.
#include "bc_internal.h"
#include "bc_wave.h"

namespace bcx {
namespace {

constexpr int32_t kPatch[3] = {16, 128, 1024};
// hops a patch may grow: enough for nearly every seed's reach on a plane
constexpr int kPatchHops[3] = {12, 26, 64};
constexpr int kScanBlock = 1024;

__device__ __forceinline__ uint32_t mix(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    return x ^ (x >> 16);
}

// Every `patch`-th vertex (by a hash) is its own patch's seed, the rest in none.
__global__ void k_lay_seeds(int32_t n, uint32_t patch, int32_t *label) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
        label[v] = mix((uint32_t)v) % patch == 0 ? v : -1;
}

// One hop: a vertex in no patch joins that of its first neighbour in one.
__global__ void k_lay_grow(int32_t n, const int32_t *row_ptr, const int32_t *col,
                           const int32_t *from, int32_t *to) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        int32_t l = from[v];
        for (int32_t e = row_ptr[v], re = row_ptr[v + 1]; l < 0 && e < re; ++e) l = from[col[e]];
        to[v] = l;
    }
}

// Vertices that no seed reached are patches of their own; the smallest
// patches' sizes.
__global__ void k_lay_count(int32_t n, int32_t *label, int32_t *size) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        if (label[v] < 0) label[v] = v;
        atomicAdd(&size[label[v]], 1);
    }
}

// The patches `inner` (seed v: inner[v] == v) lie in their seeds' patches
// `outer` (or are such patches themselves): their places there, which replace
// their sizes, and the outer patches' sizes.
__global__ void k_lay_nest(int32_t n, const int32_t *inner, int32_t *size, int32_t *outer,
                           int32_t *total) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        if (inner[v] != v || size[v] == 0) continue;
        if (outer[v] < 0) outer[v] = v;
        size[v] = atomicAdd(&total[outer[v]], size[v]);
    }
}

// x[i] becomes the sum of the entries before it among a block's `span`; the
// block's total goes to part[block], or to x[n] where one block takes all.
constexpr int kScanPer = 16, kScanSpan = kScanBlock * kScanPer;
__global__ __launch_bounds__(kScanBlock) void k_lay_scan(int32_t n, int32_t span, int32_t *x,
                                                         int32_t *part) {
    constexpr int kWaves = kScanBlock / kWave;
    __shared__ uint32_t wave_sum[kWaves];
    const int t = threadIdx.x, wave = t / kWave;
    const int32_t from = blockIdx.x * span, to = min(n, from + span);
    uint32_t carry = 0;
    for (int32_t a = from; a < to; a += kScanSpan) {
        const int32_t b = a + t * kScanPer;
        uint32_t y[kScanPer], mine = 0;
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            y[j] = b + j < to ? (uint32_t)x[b + j] : 0u;
            mine += y[j];
        }
        uint32_t sum;
        uint32_t run = wave_excl_scan(mine, sum);
        if (lane_id() == 0) wave_sum[wave] = sum;
        __syncthreads();
        uint32_t all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w == wave) run += carry + all;
            all += wave_sum[w];
        }
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            if (b + j < to) x[b + j] = (int32_t)run;
            run += y[j];
        }
        carry += all;
        __syncthreads();
    }
    if (t == 0) (part ? part[blockIdx.x] : x[n]) = (int32_t)carry;
}

// The blocks' own scans of x put together: part holds the sums before them and,
// behind those, the total.
__global__ void k_lay_add(int32_t n, int32_t parts, int32_t *x, const int32_t *part) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += gridDim.x * blockDim.x)
        x[i] = i < n ? x[i] + part[i / kScanSpan] : part[parts];
}

// pos[v]: v's place (its patches' places added up); its degree and its
// caller id there.
__global__ void k_lay_place(int32_t n, const int32_t *row_ptr, const int32_t *iperm,
                            const int32_t *l0, const int32_t *l1, const int32_t *l2,
                            int32_t *at0, const int32_t *at1, const int32_t *base, int32_t *pos,
                            int32_t *degree, int32_t *caller) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const int32_t a = l0[v], b = l1[a], c = l2[b];
        const int32_t p = base[c] + at1[b] + atomicAdd(&at0[a], 1);
        pos[v] = p;
        degree[p] = row_ptr[v + 1] - row_ptr[v];
        caller[p] = iperm[v];
    }
}

// The rows in the new order, and each vertex's first four arcs (-1: none; a
// vertex of more has kMoreArcs first, and is looked up in its row).
__global__ void k_lay_arcs(int32_t n, const int32_t *row_ptr, const int32_t *col,
                           const int32_t *pos, const int32_t *new_rp, int32_t *new_col,
                           int4 *four) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const int32_t a = row_ptr[v], d = row_ptr[v + 1] - a, p = pos[v], to = new_rp[p];
        int32_t f[4] = {-1, -1, -1, -1};
        for (int32_t j = 0; j < d; ++j) {
            const int32_t w = pos[col[a + j]];
            new_col[to + j] = w;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (j == u) f[u] = w;
        }
        four[p] = make_int4(d > 4 ? kMoreArcs : f[0], f[1], f[2], f[3]);
    }
}

__global__ void k_lay_zero(int32_t n, int32_t *x) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        x[i] = 0;
}

}  // namespace

hipError_t layout_build(const LayoutDev &d, hipStream_t stream) {
    const int32_t n = d.n;
    const dim3 grid((unsigned)std::min<int64_t>(((int64_t)n + kBlock - 1) / kBlock, 4096)),
        block(kBlock);
    int32_t *label[3], *size[3];  // size[2] becomes the largest patches' places
    for (int l = 0; l < 3; ++l) {
        // a patch grows a hop per launch
        int32_t *a = d.tmp[2 * l], *b = d.tmp[2 * l + 1];
        hipLaunchKernelGGL(k_lay_seeds, grid, block, 0, stream, n, (uint32_t)kPatch[l], a);
        for (int r = 0; r < kPatchHops[l]; ++r) {
            hipLaunchKernelGGL(k_lay_grow, grid, block, 0, stream, n, d.row_ptr, d.col_idx, a, b);
            std::swap(a, b);
        }
        label[l] = a;
        size[l] = b;
        hipLaunchKernelGGL(k_lay_zero, grid, block, 0, stream, n, b);
    }
    hipLaunchKernelGGL(k_lay_count, grid, block, 0, stream, n, label[0], size[0]);
    hipLaunchKernelGGL(k_lay_nest, grid, block, 0, stream, n, label[0], size[0], label[1], size[1]);
    hipLaunchKernelGGL(k_lay_nest, grid, block, 0, stream, n, label[1], size[1], label[2], size[2]);
    // (one block alone took 0.9 ms for a scan of 1M entries)
    auto scan = [&](int32_t *x, int32_t *part) {
        const int32_t parts = (n + kScanSpan - 1) / kScanSpan;
        hipLaunchKernelGGL(k_lay_scan, dim3(parts), dim3(kScanBlock), 0, stream, n, kScanSpan, x,
                           part);
        hipLaunchKernelGGL(k_lay_scan, dim3(1), dim3(kScanBlock), 0, stream, parts, parts, part,
                           nullptr);
        hipLaunchKernelGGL(k_lay_add, grid, block, 0, stream, n, parts, x, part);
    };
    scan(size[2], d.pos);  // (pos is written after it)
    hipLaunchKernelGGL(k_lay_place, grid, block, 0, stream, n, d.row_ptr, d.iperm, label[0],
                       label[1], label[2], size[0], size[1], size[2], d.pos, d.new_rp, d.caller);
    scan(d.new_rp, label[0]);  // (the labels have been read)
    hipLaunchKernelGGL(k_lay_arcs, grid, block, 0, stream, n, d.row_ptr, d.col_idx, d.pos,
                       d.new_rp, d.new_col, d.four);
    return hipGetLastError();
}

}  // namespace bcx
