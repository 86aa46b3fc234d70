// batch_kernels.hip -- uneven batches of Monte-Carlo requests in one
// persistent launch (the paper's dry-run workload: many bettors each asking
// for their own simulations of the race in play, Sections 3 and 6).
//
// batch_mc_kernel: one persistent launch for the whole batch (a second one
// for races with a time term of R, the paced variant), grid sized to the
// resident capacity of the GPU; every wave repeatedly takes the next work
// item from a global atomic counter (one atomic per item, issued by lane
// 0), runs that item's simulations one generation of 64 at a time with the
// template instance of its competitor count and the race's parameters in
// its LDS records, and flushes the item's wins with one 64-bit atomic per
// competitor (items shared by requests: one per simulation, to its request's
// row).  Items are ordered by expected work, largest first, so the
// smallest work ends the queue.
#include "batch_mc.hpp"
#include "kernels.hpp"
#include "race_sim.hpp"

#include <utility>

namespace bbe {

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, uint32_t v, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// probs[r][c] = wins[r][c] / sum_c wins[r][c] for c < n_r (1/n_r if the row
// is empty), 0 for the padding columns.
__global__ void batch_probs_kernel(const unsigned long long* __restrict__ wins,
                                   const ReqDesc* __restrict__ reqs, int n_reqs,
                                   double* __restrict__ probs) {
    // 64-bit index: n_reqs * 20 may exceed 2^31
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t r = i / kMaxN;
    const int c = (int)(i - r * kMaxN);
    if (r >= (size_t)n_reqs) return;
    const int n = reqs[r].rc.n;
    const unsigned long long* row = wins + r * kMaxN;
    unsigned long long tot = 0;
    for (int k = 0; k < n; ++k) tot += row[k];
    double p = 0.0;
    if (c < n) p = tot ? (double)row[c] / (double)tot : 1.0 / (double)n;
    probs[r * kMaxN + c] = p;
}

// ---------------------------------------------------------------- launchers

hipError_t launch_batch_mc(const BatchArgs& a, int waves_per_block, int grid, bool paced,
                           hipStream_t s) {
    if (waves_per_block != 1 && waves_per_block != 2 && waves_per_block != 4)
        return hipErrorInvalidValue;
    if (paced) return launch_batch_mc_paced(a, waves_per_block, grid, s);
    hipLaunchKernelGGL((batch_mc_kernel<false>), dim3(grid), dim3(64 * waves_per_block),
                       waves_per_block * kWaveBytes, s, a);
    return hipGetLastError();
}

int batch_blocks_per_cu(int waves_per_block, bool paced) {
    if (waves_per_block < 1 || waves_per_block > 4) return 1;
    if (paced) return batch_blocks_per_cu_paced(waves_per_block);
    static int cache[5] = {};
    int& c = cache[waves_per_block];
    if (!c) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_mc_kernel<false>,
                                                         64 * waves_per_block,
                                                         waves_per_block * kWaveBytes) !=
                hipSuccess ||
            nb < 1)
            nb = 1;
        c = nb;
    }
    return c;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_batch_probs(const unsigned long long* wins, const ReqDesc* reqs, int n_reqs,
                              double* probs, hipStream_t s) {
    long total = (long)n_reqs * kMaxN;
    hipLaunchKernelGGL(batch_probs_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                       wins, reqs, n_reqs, probs);
    return hipGetLastError();
}

}  // namespace bbe
