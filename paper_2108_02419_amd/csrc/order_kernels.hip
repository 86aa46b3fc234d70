// order_kernels.hip -- tallies over finish orders (paper Section 6: the
// finish orders of repeated seeded runs estimate a probability mass function
// over the n! possible orders; Section 3: a bettor's view of a race is a set
// of such frequentist estimates).
//
// rank_counts_kernel: counts[c][r] += 1 for every simulation in which
// competitor c finished at rank r (finish-position / place probabilities).
// order_pmf_kernel (n <= 7): counts[lexicographic rank of the order] += 1
// for every simulation whose order is complete.
//
// Both tally in LDS and flush with one 64-bit atomic per non-zero bin.  What
// bounds them is not the matrix (n bytes a simulation, read once) but the
// tally: the lanes of a wave mostly hit the few bins of the likely orders, and
// LDS adds to one address go one by one, as do the flush's adds to one address
// of memory.  So each bin has up to kCopies copies, a lane adds to the one of
// its index (64 lanes, at most two of them on one address), and one large
// workgroup per CU leaves few flushes: 10^6 orders of 20 with the clearing of
// the counts, 55.7 us with one copy and 2048 workgroups, 13.5 us so (1.5 TB/s).
#include "kernels.hpp"

namespace bbe {

constexpr int kOrdBlock = 1024;
constexpr int kCopies = 32;  // of a bin, at most

// Sums the copies of bin i (each lane starting at another copy: no two lanes
// of a wave on one bank).
__device__ __forceinline__ uint32_t bin_sum(const uint32_t* bins, int i, int copies) {
    uint32_t v = 0u;
    for (int k = 0; k < copies; ++k) v += bins[i * copies + ((k + i) & (copies - 1))];
    return v;
}

// The matrix as a stream of bytes: byte i is rank i mod n of simulation i / n.
// A thread takes 16 aligned bytes at a time (any n, any address; the bytes
// before the first and after the last aligned 16 go to one thread each).
__global__ void __launch_bounds__(kOrdBlock)
    rank_counts_kernel(const uint8_t* __restrict__ orders, uint32_t n_sims, int n,
                       unsigned long long* __restrict__ counts) {
    __shared__ uint32_t bins[kMaxN * kMaxN * kCopies];
    for (int i = threadIdx.x; i < n * n * kCopies; i += kOrdBlock) bins[i] = 0u;
    __syncthreads();
    const uint32_t copy = threadIdx.x & (kCopies - 1);
    const uint64_t bytes = (uint64_t)n_sims * (uint32_t)n;
    const uint64_t lead = (0u - (uint32_t)reinterpret_cast<uintptr_t>(orders)) & 15u;
    const uint64_t head = lead < bytes ? lead : bytes;
    const uint64_t blocks = (bytes - head) >> 4;
    const uint64_t gid = (uint64_t)blockIdx.x * kOrdBlock + threadIdx.x;
    auto tally = [&](uint32_t c, uint32_t r) {
        if (c < (uint32_t)n) atomicAdd(&bins[(c * n + r) * kCopies + copy], 1u);
    };
    const uint64_t stride = (uint64_t)gridDim.x * kOrdBlock;
    // the rank of a thread's next 16 bytes without a division each time
    uint32_t r0 = (uint32_t)((head + (gid << 4)) % (uint32_t)n);
    const uint32_t step = (uint32_t)((stride << 4) % (uint32_t)n);
    for (uint64_t b = gid; b < blocks; b += stride) {
        const uint4 v = *reinterpret_cast<const uint4*>(orders + head + (b << 4));
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t r = r0;
        r0 += step;
        r0 = r0 >= (uint32_t)n ? r0 - n : r0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            tally((w[j >> 2] >> (8 * (j & 3))) & 0xFFu, r);
            r = r + 1 == (uint32_t)n ? 0u : r + 1;
        }
    }
    const uint64_t rest = bytes - (blocks << 4);  // head bytes, then the last ones (< 32)
    if (gid < rest) {
        const uint64_t at = gid < head ? gid : (blocks << 4) + gid;
        tally(orders[at], (uint32_t)(at % (uint32_t)n));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n * n; i += kOrdBlock) {
        const uint32_t v = bin_sum(bins, i, kCopies);
        if (v) atomicAdd(&counts[i], (unsigned long long)v);
    }
}

// Lexicographic rank of a complete order (its Lehmer code read in the
// factorial number system); -1 if some rank is unfilled (0xFF) or holds an
// index >= n.
template <int N>
__device__ __forceinline__ int lex_rank(const uint32_t (&row)[N]) {
    int rank = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (row[i] >= (uint32_t)N) return -1;
        int smaller = 0;
#pragma unroll
        for (int j = i + 1; j < N; ++j) smaller += (row[j] < row[i]) ? 1 : 0;
        rank = rank * (N - i) + smaller;
    }
    return rank;
}

// Copies of each of the n! bins: as many as 40 KB hold.
constexpr int pmf_copies(int n) { return n <= 5 ? kCopies : n == 6 ? 8 : 2; }

template <int N>
__global__ void __launch_bounds__(kOrdBlock)
    order_pmf_kernel(const uint8_t* __restrict__ orders, uint32_t n_sims, int n_fact,
                     unsigned long long* __restrict__ counts) {
    constexpr int C = pmf_copies(N);
    extern __shared__ uint32_t bins[];  // [n!][C]
    for (int i = threadIdx.x; i < n_fact * C; i += kOrdBlock) bins[i] = 0u;
    __syncthreads();
    const uint32_t copy = threadIdx.x & (C - 1);
    const uint64_t stride = (uint64_t)gridDim.x * kOrdBlock;
    for (uint64_t s = (uint64_t)blockIdx.x * kOrdBlock + threadIdx.x; s < n_sims; s += stride) {
        uint32_t row[N];
#pragma unroll
        for (int r = 0; r < N; ++r) row[r] = orders[s * (uint64_t)N + r];
        const int k = lex_rank<N>(row);
        if (k >= 0) atomicAdd(&bins[k * C + copy], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n_fact; i += kOrdBlock) {
        const uint32_t v = bin_sum(bins, i, C);
        if (v) atomicAdd(&counts[i], (unsigned long long)v);
    }
}

// Workgroups for `items` thread-loads: one per CU at most.
static int order_grid(uint64_t items) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const uint64_t want = (items + kOrdBlock - 1) / kOrdBlock;
    return (int)(want < 1 ? 1 : (want < (uint64_t)cus ? want : (uint64_t)cus));
}

hipError_t launch_rank_counts(const uint8_t* orders, uint32_t n_sims, int n,
                              unsigned long long* counts, hipStream_t s) {
    hipError_t e = launch_zero_u64(counts, n * n, s);
    if (e != hipSuccess || n_sims == 0) return e;
    // a grid for the 16-byte blocks, and of 32 threads at least for the rest
    hipLaunchKernelGGL(rank_counts_kernel, dim3(order_grid(((uint64_t)n_sims * n) >> 4)),
                       dim3(kOrdBlock), 0, s, orders, n_sims, n, counts);
    return hipGetLastError();
}

template <int N>
static hipError_t launch_pmf_n(const uint8_t* orders, uint32_t n_sims, int n_fact,
                               unsigned long long* counts, hipStream_t s) {
    hipLaunchKernelGGL(order_pmf_kernel<N>, dim3(order_grid(n_sims)), dim3(kOrdBlock),
                       n_fact * pmf_copies(N) * sizeof(uint32_t), s, orders, n_sims, n_fact,
                       counts);
    return hipGetLastError();
}

hipError_t launch_order_pmf(const uint8_t* orders, uint32_t n_sims, int n, int n_fact,
                            unsigned long long* counts, hipStream_t s) {
    hipError_t e = launch_zero_u64(counts, n_fact, s);
    if (e != hipSuccess || n_sims == 0) return e;
    switch (n) {
        case 1: return launch_pmf_n<1>(orders, n_sims, n_fact, counts, s);
        case 2: return launch_pmf_n<2>(orders, n_sims, n_fact, counts, s);
        case 3: return launch_pmf_n<3>(orders, n_sims, n_fact, counts, s);
        case 4: return launch_pmf_n<4>(orders, n_sims, n_fact, counts, s);
        case 5: return launch_pmf_n<5>(orders, n_sims, n_fact, counts, s);
        case 6: return launch_pmf_n<6>(orders, n_sims, n_fact, counts, s);
        case 7: return launch_pmf_n<7>(orders, n_sims, n_fact, counts, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bbe
