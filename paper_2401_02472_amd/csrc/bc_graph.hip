// Graph set-up kernels: relabelling of the CSR into the library's internal
// vertex order, and gathers from internal order back to the caller's order.
#include "bc_internal.h"

namespace bcx {
namespace {

__global__ __launch_bounds__(kBlock) void k_relabel(int32_t n, int64_t nnz,
                                                    const int32_t *old_rp,
                                                    const int32_t *old_ci,
                                                    const int32_t *new_rp,
                                                    const int32_t *perm,
                                                    const int32_t *iperm, int32_t *new_ci) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += stride) {
        // owner u: last vertex with new_rp[u] <= e
        int32_t lo = 0, hi = n - 1;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo + 1) / 2;
            if ((int64_t)new_rp[mid] <= e) lo = mid;
            else hi = mid - 1;
        }
        const int32_t o = iperm[lo];
        new_ci[e] = perm[old_ci[(int64_t)old_rp[o] + (e - new_rp[lo])]];
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_gather(int32_t n, const int32_t *perm, const T *src,
                                                   T *dst) {
    for (int32_t o = blockIdx.x * blockDim.x + threadIdx.x; o < n; o += gridDim.x * blockDim.x)
        dst[o] = src[perm[o]];
}

// Four breadth-first searches at once, a byte each of a vertex's word: 0 not
// reached, else level + 1.
__global__ __launch_bounds__(kBlock) void k_probe_seed(int32_t n, int32_t live, int32_t steps,
                                                       uint32_t *word, int32_t *found) {
    const int32_t at = blockIdx.x * blockDim.x + threadIdx.x, all = gridDim.x * blockDim.x;
    for (int32_t v = at; v < n; v += all) {
        uint32_t x = 0;
        for (int j = 0; j < 4; ++j)
            if (v == (int32_t)((int64_t)live * j / 4)) x |= 1u << (8 * j);
        word[v] = x;
    }
    for (int32_t i = at; i < steps + 4; i += all) found[i] = 0;
}

// Level L + 1 of the four: a vertex takes it where a neighbour is at level L.
// Only a vertex's own thread writes its word, and a value that appears while
// others read it is no level L.
__global__ __launch_bounds__(kBlock) void k_probe_step(int32_t n, int32_t L, const int32_t *rp,
                                                       const int32_t *ci, uint32_t *word,
                                                       int32_t *found) {
    if (L > 0 && found[L - 1] == 0) return;
    bool any = false;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const uint32_t mine = word[v];
        uint32_t take = 0;
        bool open = false;
        for (int j = 0; j < 4; ++j) open |= (mine >> (8 * j) & 255u) == 0u;
        if (!open) continue;
        for (int32_t e = rp[v], re = rp[v + 1]; e < re; ++e) {
            const uint32_t x = word[ci[e]];
            for (int j = 0; j < 4; ++j)
                if ((mine >> (8 * j) & 255u) == 0u && (x >> (8 * j) & 255u) == (uint32_t)L + 1u)
                    take |= ((uint32_t)L + 2u) << (8 * j);
        }
        if (take) {
            word[v] = mine | take;
            any = true;
        }
    }
    if (any) found[L] = 1;
}

// count[j] += vertices that search j has reached.
__global__ __launch_bounds__(kBlock) void k_probe_count(int32_t n, const uint32_t *word,
                                                        int32_t *count) {
    int32_t mine[4] = {};
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
        for (int j = 0; j < 4; ++j) mine[j] += (word[v] >> (8 * j) & 255u) != 0u;
    __shared__ int32_t sum[4];
    if (threadIdx.x < 4) sum[threadIdx.x] = 0;
    __syncthreads();
    for (int j = 0; j < 4; ++j)
        if (mine[j]) atomicAdd(&sum[j], mine[j]);
    __syncthreads();
    if (threadIdx.x < 4 && sum[threadIdx.x]) atomicAdd(&count[threadIdx.x], sum[threadIdx.x]);
}

int grid_for(int64_t items) {
    int64_t g = (items + kBlock - 1) / kBlock;
    return (int)(g < 1 ? 1 : (g > 4096 ? 4096 : g));
}

}  // namespace

hipError_t relabel_csr(int32_t n, int64_t nnz, const int32_t *old_rp, const int32_t *old_ci,
                       const int32_t *new_rp, const int32_t *perm, const int32_t *iperm,
                       int32_t *new_ci, hipStream_t stream) {
    if (nnz == 0 || n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_relabel, dim3(grid_for(nnz)), dim3(kBlock), 0, stream, n, nnz, old_rp,
                       old_ci, new_rp, perm, iperm, new_ci);
    return hipGetLastError();
}

hipError_t depth_probe(int32_t n, int32_t live, const int32_t *row_ptr, const int32_t *col_idx,
                       int32_t steps, uint32_t *word, int32_t *found, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_probe_seed, dim3(grid_for(n)), dim3(kBlock), 0, stream, n, live, steps,
                       word, found);
    for (int32_t L = 0; L < steps; ++L)
        hipLaunchKernelGGL(k_probe_step, dim3(grid_for(n)), dim3(kBlock), 0, stream, n, L, row_ptr,
                           col_idx, word, found);
    hipLaunchKernelGGL(k_probe_count, dim3(std::min(grid_for(n), 512)), dim3(kBlock), 0, stream, n,
                       word, found + steps);
    return hipGetLastError();
}

hipError_t gather_f64(int32_t n, const int32_t *perm, const double *src, double *dst,
                      hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather<double>, dim3(grid_for(n)), dim3(kBlock), 0, stream, n, perm,
                       src, dst);
    return hipGetLastError();
}

// out[v] = (accumulate ? out[v] : 0) + parts[0][v] + parts[1][v] + ... (in
// part order), parts stored [nparts][n].
__global__ void k_sum_parts(int32_t n, const double *parts, int32_t nparts, double *out,
                            int32_t accumulate) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        double t = accumulate ? out[v] : 0.0;
        for (int32_t i = 0; i < nparts; ++i) t += parts[(size_t)i * n + v];
        out[v] = t;
    }
}

hipError_t sum_parts(int32_t n, const double *parts, int32_t nparts, double *out,
                     hipStream_t stream, bool accumulate) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_sum_parts, dim3(grid_for(n)), dim3(kBlock), 0, stream, n, parts, nparts,
                       out, accumulate ? 1 : 0);
    return hipGetLastError();
}

hipError_t gather_i32(int32_t n, const int32_t *perm, const int32_t *src, int32_t *dst,
                      hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather<int32_t>, dim3(grid_for(n)), dim3(kBlock), 0, stream, n, perm,
                       src, dst);
    return hipGetLastError();
}

}  // namespace bcx
