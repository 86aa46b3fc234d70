// bettor_kernels.hip -- the in-play side of the model on gfx950: the views of
// the cheap bettor rules of paper Section 5 (LinEx, LW, UD, ZI) over the
// trace of the race that bettors watch.
//
// bettor_views_kernel: a workgroup forms the views of some slices of 1024
// bettors, each grouped by kind so that nearly every wave runs a single rule,
// at chunks of kViewRowsPerBlock trace rows.  Per chunk it stages the rows in
// LDS -- with up to kViewWindow rows of history before them where there are
// LinEx bettors -- and settles everything that does not depend on the bettor
// once: each row's leader and runner-up, and LinEx's pick for every window up
// to the longest.
// A bettor's view is then a look-up:
//   LW     the leader (ties to the lowest index);
//   UD     the runner-up while fl(x_P1 - x_P2) < D, else the leader;
//   LinEx  over a window w = min(N, r) ticks, the competitor with the least
//          remaining distance fl(L - x) per displacement fl(x - x_back),
//          among those that moved; the two ratios are compared exactly by
//          cross-multiplying in double precision (products of two floats
//          are exact there); with w = 0 or nobody moving, the leader (windows
//          longer than kViewPicks: a scan per bettor);
//   ZI     a uniform competitor, floor(w * n / 2^32) for the first word w
//          of the Philox block with counter (t, bettor, ~0, ~0).
// The views go to memory through LDS, in the caller's order and 16 bytes at a
// time; ZI's and LinEx's tallies have 16 copies of each bin in LDS, since most
// bettors back the same few competitors, and the others' are counted by wave.
// (With a scan per LinEx bettor, byte stores and one copy of the bins, 10^5
// bettors took 140 us for 240 rows of a 20-competitor race, 46 us so; what is
// left is ZI's Philox rounds and the 24 MB of views.)
#include "bettors.hpp"
#include "race_sim.hpp"

#include <utility>

namespace bbe {

// LinEx pick over rows x (now) and back (w ticks earlier): least
// fl(L - x_c) / fl(x_c - back_c) among positive displacements, compared
// exactly; -1 if nobody moved.
__device__ __forceinline__ int linex_scan(const float* __restrict__ x,
                                          const float* __restrict__ back, int n, float L) {
    int best = -1;
    float bre = 0.0f, bdi = 1.0f;
#pragma unroll 4
    for (int c = 0; c < n; ++c) {
        const float xc = x[c];
        const float disp = xc - back[c];
        const float rem = L - xc;
        const bool better = disp > 0.0f && (best < 0 || (double)rem * (double)bdi <
                                                            (double)bre * (double)disp);
        best = better ? c : best;
        bre = better ? rem : bre;
        bdi = better ? disp : bdi;
    }
    return best;
}

// Leader and runner-up (the leader where n = 1) of a row that holds NaN, as a
// scan finds them: a NaN is passed by nobody and passes nobody.
__device__ __forceinline__ void scan_row(const float* x, int n, int& p1, int& p2) {
    p1 = 0;
    for (int c = 1; c < n; ++c)
        if (x[c] > x[p1]) p1 = c;
    p2 = -1;
    for (int c = 0; c < n; ++c)
        if (c != p1 && (p2 < 0 || x[c] > x[p2])) p2 = c;
    if (p2 < 0) p2 = p1;
}

constexpr int kViewThreads = 256;
constexpr int kViewEach = kViewSlice / kViewThreads;
constexpr int kViewCopies = 16;
constexpr uint32_t kViewGroups = 5 * 256;

__global__ void __launch_bounds__(kViewThreads)
    __attribute__((amdgpu_waves_per_eu(5))) bettor_views_kernel(const ViewArgs a) {
    constexpr int R = kViewRowsPerBlock;
    constexpr int kStride = kMaxN + 1;  // of a staged row: odd, to spread the banks
    __shared__ float s_rows[(kViewWindow + R) * kStride];
    __shared__ uint32_t s_cnt[R * kMaxN * kViewCopies];
    __shared__ int s_p1[R], s_p2[R];    // leader, runner-up (the leader where n = 1)
    __shared__ float s_x1[R], s_x2[R];  // their positions
    __shared__ uint8_t s_pick[R][kViewPicks];  // LinEx's pick at window w + 1
    // views in the caller's order, each row placed as in memory modulo 16
    __shared__ __attribute__((aligned(16))) uint8_t s_view[R][kViewSlice + 16];
    const int n = a.n;
    const uint32_t copy = threadIdx.x & (kViewCopies - 1);
    const int hist = (int)min(a.window, (uint32_t)kViewWindow);
    const int picks = (int)min(a.window, (uint32_t)kViewPicks);
    const uint32_t begin = blockIdx.x * a.slices * kViewSlice;
    const uint32_t end =
        (uint32_t)min((uint64_t)begin + (uint64_t)a.slices * kViewSlice, (uint64_t)a.n_bettors);

    for (uint32_t i0 = blockIdx.y * a.rows; i0 < a.n_eval; i0 += gridDim.y * a.rows) {
        const int nr = (int)min(a.rows, a.n_eval - i0);
        const uint32_t r0 = a.first_row + i0;
        // rows lo .. r0 + nr - 1 in LDS: the chunk and the history before it
        const uint32_t lo = r0 > (uint32_t)hist ? r0 - hist : 0u;
        const int nstage = (int)(r0 - lo + nr) * n;
        const float* __restrict__ src = a.trace + (size_t)lo * n;
        for (int k = threadIdx.x; k < nstage; k += kViewThreads)
            s_rows[(k / n) * kStride + k % n] = src[k];
        for (int k = threadIdx.x; k < nr * n * kViewCopies; k += kViewThreads) s_cnt[k] = 0u;
        __syncthreads();
        // a thread for each row and competitor: the leader has nobody before
        // it in (position, lowest index) order, the runner-up one; NaN has no
        // place in that order, so a row with one is scanned
        for (int k = threadIdx.x; k < nr * n; k += kViewThreads) {
            const int ii = k / n, c = k - ii * n;
            const float* x = s_rows + ((int)(r0 - lo) + ii) * kStride;
            const float xc = x[c];
            int before = 0;
            bool nan = false;
#pragma unroll 4
            for (int j = 0; j < n; ++j) {
                before += x[j] > xc || (x[j] == xc && j < c);
                nan |= x[j] != x[j];
            }
            if (nan) {
                int p1, p2;
                if (c == 0) {
                    scan_row(x, n, p1, p2);
                    s_p1[ii] = p1;
                    s_x1[ii] = x[p1];
                    s_p2[ii] = p2;
                    s_x2[ii] = x[p2];
                }
                continue;
            }
            if (before == 0) {
                s_p1[ii] = c;
                s_x1[ii] = xc;
            }
            if (before == 1 || n == 1) {
                s_p2[ii] = c;
                s_x2[ii] = xc;
            }
        }
        // LinEx's views, a thread for each row and window
        for (int k = threadIdx.x; k < nr * picks; k += kViewThreads) {
            const int ii = k / picks, w = k - ii * picks + 1;
            const int at = (int)(r0 - lo) + ii;
            const float* x = s_rows + at * kStride;
            // 0xFF: the leader (no such row, or nobody moved)
            int v = 0xFF;
            if (w <= at)
                v = linex_scan(x, x - w * kStride, n, a.L);
            else if ((uint32_t)w <= r0 + ii)
                v = linex_scan(x, a.trace + (size_t)(r0 + ii - w) * n, n, a.L);
            s_pick[ii][w - 1] = (uint8_t)v;
        }
        __syncthreads();

        for (uint32_t first = begin; first < end; first += kViewSlice) {
            const uint32_t count = min((uint32_t)kViewSlice, end - first);
            // where a row's views begin in s_view
            const uint32_t at0 = (uint32_t)reinterpret_cast<uintptr_t>(a.views) +
                                 (uint32_t)((size_t)i0 * a.n_bettors + first);
            auto put = [&](int ii, uint32_t local, int v) {
                s_view[ii][((at0 + (uint32_t)ii * a.n_bettors) & 15u) + local] = (uint8_t)v;
            };
            // counts of the wave's bettors that back competitor v
            auto tally = [&](int ii, int v, uint64_t who) {
                if (__lane_id() == (uint32_t)__builtin_ctzll(who | (1ull << 63)))
                    atomicAdd(&s_cnt[(ii * n + v) * kViewCopies + copy],
                              (uint32_t)__popcll(who));
            };
            uint8_t kinds[kViewEach];
            uint32_t ids[kViewEach];
            float params[kViewEach];
#pragma unroll
            for (int q = 0; q < kViewEach; ++q) {
                const uint32_t j = min(q * kViewThreads + threadIdx.x, count - 1u);
                kinds[q] = a.kind[first + j];
                ids[q] = a.id[first + j];
                params[q] = a.param[first + j];
            }
#pragma unroll
            for (int q = 0; q < kViewEach; ++q) {
                if (q * kViewThreads + threadIdx.x >= count) continue;
                const uint8_t kind = kinds[q];
                const uint32_t id = ids[q], local = id - first;
                const float param = params[q];
                if (kind == kZI) {
                    for (int ii = 0; ii < nr; ++ii) {
                        const U4 w = philox4x32_10(a.t0 + r0 + ii, id, 0xFFFFFFFFu, 0xFFFFFFFFu,
                                                   a.k0, a.k1);
                        const int v = (int)(((uint64_t)w.x * (uint32_t)n) >> 32);
                        put(ii, local, v);
                        atomicAdd(&s_cnt[(ii * n + v) * kViewCopies + copy], 1u);
                    }
                } else if (kind == kLinEx) {
                    const uint32_t window = (uint32_t)param;
                    for (int ii = 0; ii < nr; ++ii) {
                        const uint32_t r = r0 + ii, w = min(window, r);
                        int v = 0xFF;
                        if (w - 1 < (uint32_t)picks)
                            v = s_pick[ii][w - 1];
                        else if (w > 0)
                            v = linex_scan(s_rows + (r - lo) * kStride,
                                           a.trace + (size_t)(r - w) * n, n, a.L) & 0xFF;
                        v = v == 0xFF ? s_p1[ii] : v;
                        put(ii, local, v);
                        atomicAdd(&s_cnt[(ii * n + v) * kViewCopies + copy], 1u);
                    }
                } else if (kind == kUD) {
                    const float dist = param;
                    for (int ii = 0; ii < nr; ++ii) {
                        const bool second = s_x1[ii] - s_x2[ii] < dist;
                        const int p1 = s_p1[ii], p2 = s_p2[ii];
                        put(ii, local, second ? p2 : p1);
                        const uint64_t w2 = __builtin_amdgcn_ballot_w64(second);
                        const uint64_t w1 = __builtin_amdgcn_ballot_w64(!second);
                        if (w2) tally(ii, p2, w2);
                        if (w1) tally(ii, p1, w1);
                    }
                } else {
                    const uint64_t all = __builtin_amdgcn_ballot_w64(true);
                    for (int ii = 0; ii < nr; ++ii) {
                        const int p1 = s_p1[ii];
                        put(ii, local, p1);
                        tally(ii, p1, all);
                    }
                }
            }
            __syncthreads();
            if (a.views) {
                for (int ii = threadIdx.x >> 6; ii < nr; ii += kViewThreads / 64) {
                    uint8_t* dst = a.views + (size_t)(i0 + ii) * a.n_bettors + first;
                    const uint32_t pad = (uint32_t)reinterpret_cast<uintptr_t>(dst) & 15u;
                    const uint32_t stop = pad + count;
                    // 16-byte pieces of [pad, stop); the first and last may be partial
                    for (uint32_t k = 16u * (threadIdx.x & 63); k < stop; k += 16u * 64u) {
                        if (k >= pad && k + 16u <= stop) {
                            *reinterpret_cast<uint4*>(dst - pad + k) =
                                *reinterpret_cast<const uint4*>(&s_view[ii][k]);
                        } else {
                            for (uint32_t b = max(k, pad); b < min(k + 16u, stop); ++b)
                                dst[b - pad] = s_view[ii][b];
                        }
                    }
                }
                __syncthreads();
            }
        }
        if (a.counts)
            for (int k = threadIdx.x; k < nr * n; k += kViewThreads) {
                uint32_t v = 0u;
                for (int j = 0; j < kViewCopies; ++j)
                    v += s_cnt[k * kViewCopies + ((j + k) & (kViewCopies - 1))];
                if (v) atomicAdd(&a.counts[(size_t)i0 * n + k], v);
            }
        __syncthreads();
    }
}

// RP(d) views: the competitor with the most dry-run wins (lowest index on
// ties), one thread per bettor row of the win-count matrix.
constexpr int kRpBlock = 256;

__global__ void __launch_bounds__(kRpBlock)
    rp_views_kernel(const unsigned long long* __restrict__ wins, uint32_t n_bettors, int n,
                    int stride, uint8_t* __restrict__ views, uint32_t* __restrict__ counts) {
    __shared__ uint32_t s_cnt[kMaxN];
    if ((int)threadIdx.x < n) s_cnt[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t b = blockIdx.x * kRpBlock + threadIdx.x;
    if (b < n_bettors) {
        const unsigned long long* __restrict__ row = wins + (size_t)b * stride;
        int best = 0;
        unsigned long long bw = row[0];
        for (int c = 1; c < n; ++c) {
            const unsigned long long w = row[c];
            if (w > bw) {
                bw = w;
                best = c;
            }
        }
        if (views) views[b] = (uint8_t)best;
        atomicAdd(&s_cnt[best], 1u);
    }
    __syncthreads();
    if (counts && (int)threadIdx.x < n && s_cnt[threadIdx.x])
        atomicAdd(&counts[threadIdx.x], s_cnt[threadIdx.x]);
}

__global__ void zero_u32_kernel(uint32_t* __restrict__ p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------- launchers

hipError_t launch_bettor_views(const ViewArgs& a, hipStream_t s) {
    if (a.n_eval == 0 || a.n_bettors == 0) return hipSuccess;
    if (a.counts) {
        const size_t total = (size_t)a.n_eval * a.n;
        hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                           s, a.counts, total);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint32_t slices = (a.n_bettors + kViewSlice - 1) / kViewSlice;
    ViewArgs v = a;
    // Fewer rows a workgroup where 8 would leave CUs without one.
    v.rows = kViewRowsPerBlock;
    while (v.rows > 1 && (uint64_t)slices * ((a.n_eval + v.rows - 1) / v.rows) < 512) v.rows /= 2;
    const uint64_t gy_need = ((uint64_t)a.n_eval + v.rows - 1) / v.rows;
    const unsigned gy = gy_need < 65535u ? (unsigned)gy_need : 65535u;
    // Slices share what a workgroup settles per row: as many each as it takes
    // for all workgroups to be resident at once (5 a CU: 10^5 bettors x 240
    // rows, 3 slices 990 workgroups, 46 us; 2 slices 1470, 53 us).
    const uint64_t each = ((uint64_t)slices * gy + kViewGroups - 1) / kViewGroups;
    v.slices = each < slices ? (uint32_t)each : slices;
    hipLaunchKernelGGL(bettor_views_kernel, dim3((slices + v.slices - 1) / v.slices, gy),
                       dim3(kViewThreads), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_rp_views(const unsigned long long* wins, uint32_t n_bettors, int n, int stride,
                           uint8_t* views, uint32_t* counts, hipStream_t s) {
    if (counts) {
        hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(256), 0, s, counts, (size_t)n);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_bettors == 0) return hipSuccess;
    hipLaunchKernelGGL(rp_views_kernel, dim3((n_bettors + kRpBlock - 1) / kRpBlock),
                       dim3(kRpBlock), 0, s, wins, n_bettors, n, stride, views, counts);
    return hipGetLastError();
}

}  // namespace bbe
