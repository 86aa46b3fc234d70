// batch_mc.hpp -- the persistent batch kernel template (see
// batch_kernels.hip).  Its plain variant is instantiated in
// batch_kernels.hip and its paced variant (time term of R) in
// batch_kernels_paced.hip, each in a translation unit of its own so that
// neither affects the other's code generation.
#pragma once

#include "kernels.hpp"
#include "race_sim.hpp"

#include <utility>

namespace bbe {

// Per-wave LDS: draw table [kMaxN][64] floats, parameter records, win
// histogram, the lanes' result rows, simulation indices, request ids and
// start states (u32[64] each), the start state in slot order (positions,
// previous steps, competitor ids) so that it does not occupy registers, and
// the byte table the ranking of several same-tick finishers uses.
constexpr uint32_t kWaveU = kMaxN * 256;
constexpr uint32_t kWavePar = kMaxN * 32;
constexpr uint32_t kWaveHist = 128;
constexpr uint32_t kWaveLanes = 1024;
constexpr uint32_t kWaveInit = kMaxN * 12;
constexpr uint32_t kWaveIds = kMaxN * 64;  // finisher ids of a tick, u8[N][64]
constexpr uint32_t kWaveBytes = kWaveU + kWavePar + kWaveHist + kWaveLanes + kWaveInit + kWaveIds;

__device__ __forceinline__ unsigned long long wave_sum_u64b(unsigned long long v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Parked slots stop being stepped 2 at a time once every lane has parked
// them, from N = 6 on.
template <int N>
constexpr int batch_skip_step() {
    return N >= 6 ? 2 : 0;
}

// One work item.  The simulations of an item with kChunkLanes may belong to
// several requests, all of the same race and stop_after.  They start from the
// same state unless the states were changed since the items were made: a
// generation then runs once for each state among its lanes (where that takes
// longer than items without shared lanes, the launch takes those).
// What differs by lane is read from LDS where it is used, by the items of one
// request too: a variant with scalar indices for those was 2% faster at 5
// competitors and equal or up to 2% slower from 9 on (40000 requests of 100 or
// 128 simulations), as it needed more registers around the generation.
template <int N, bool kPaced>
__device__ __forceinline__ void run_chunk(const BatchArgs& a, const Chunk& ch, char* smem,
                                          uint32_t wbase, int lane, unsigned long long& steps) {
    const ReqDesc& rq = a.reqs[ch.req];
    const bool of_one = !(ch.n & kChunkLanes);
    const uint32_t ubase = lds_addr(smem) + wbase;
    const uint32_t pbase = ubase + kWaveU;
    const uint32_t hbase = pbase + kWavePar;
    const uint32_t lbase = hbase + kWaveHist;
    const uint32_t ibase = lbase + kWaveLanes + kWaveInit;
    float* d0 = reinterpret_cast<float*>(smem + wbase + kWaveU + kWavePar + kWaveHist + kWaveLanes);
    float* s0 = d0 + kMaxN;
    uint8_t* id0 = reinterpret_cast<uint8_t*>(s0 + kMaxN);
    write_params<N>(pbase, rq.rc, lane);
    if constexpr (kPaced) write_pace<N>(pbase, rq.pace, lane);
    if (lane < N) lds_st<uint32_t>(hbase + 4u * lane, 0u);
    const StepBounds sb{rq.rc.step_cap, rq.rc.reach2, rq.rc.reach8};
    for (uint32_t g = 0; g < ch.count; g += 64) {
        const bool live = g + lane_here() < ch.count;
        {
            const uint32_t i = ch.first + (live ? g + lane_here() : 0u);
            const PackLane pl = of_one ? PackLane{ch.req, rq.sim_begin + i} : a.lanes[i];
            const uint32_t at = lbase + 4u * lane_here();
            lds_st<uint32_t>(at, pl.row);
            lds_st<uint32_t>(at + 256u, pl.sim);
            lds_st<uint32_t>(at + 512u, a.reqs[pl.row].request);
            lds_st<uint32_t>(at + 768u, a.state_of[pl.row]);
        }
        uint64_t todo = __builtin_amdgcn_ballot_w64(live);
        while (todo) {
            const uint32_t state = __builtin_amdgcn_readfirstlane(
                lds_ld<uint32_t>(lbase + 768u + 4u * (uint32_t)__builtin_ctzll(todo)));
            const bool mine = ((todo >> lane_here()) & 1ull) &&
                              lds_ld<uint32_t>(lbase + 768u + 4u * lane_here()) == state;
            todo &= ~__builtin_amdgcn_ballot_w64(mine);
            const StartState& st = a.states[state];
            if (lane < N) {
                d0[lane] = st.d0[lane];
                s0[lane] = st.s0[lane];
                id0[lane] = st.id0[lane];
            }
            // re-read the start state from LDS each time rather than keeping
            // 3N registers live across the loop
            __asm__ volatile("" ::: "memory");
            run_generation<N, kPaced ? kPaceTable : kPaceOff, batch_skip_step<N>()>(
                ubase, ibase, pbase, rq.rc.L, sb, d0, s0, id0, st.t0, mine,
                [&](uint32_t l) { return lds_ld<uint32_t>(lbase + 256u + 4u * l); },
                [&](uint32_t l) { return lds_ld<uint32_t>(lbase + 512u + 4u * l); }, a.k0, a.k1,
                rq.stop_after, kNoRow,
                [&](uint32_t c) {
                    if (of_one) {
                        atomicAdd(reinterpret_cast<uint32_t*>(smem + wbase + kWaveU + kWavePar) +
                                      c,
                                  1u);
                    } else {
                        const uint32_t row = lds_ld<uint32_t>(lbase + 4u * lane_here());
                        atomicAdd(&a.wins[(size_t)row * kMaxN + c], 1ull);
                    }
                },
                steps);
        }
    }
    if (of_one && lane < N) {
        const uint32_t w = lds_ld<uint32_t>(hbase + 4u * lane);
        if (w) atomicAdd(&a.wins[(size_t)ch.req * kMaxN + lane], (unsigned long long)w);
    }
}

// Runs a work item with the template instance of its competitor count (a
// wave-uniform switch on n).
template <bool kPaced, int... I>
__device__ __forceinline__ void run_chunk_any(int n, const BatchArgs& a, const Chunk& ch,
                                              char* smem, uint32_t wbase, int lane,
                                              unsigned long long& steps,
                                              std::integer_sequence<int, I...>) {
    (void)((n == I + 1 ? (run_chunk<I + 1, kPaced>(a, ch, smem, wbase, lane, steps), true)
                       : false) ||
           ...);
}

// The persistent kernel: one launch serves the work items of every
// competitor count (one launch for the plain races, one for the paced);
// waves take items from one global queue, ordered longest first across the
// whole batch, so that the shortest items end the launch.  Up to 4 waves per
// workgroup (blockDim.x = 64 * waves); the register budget aims at 4 waves
// per SIMD (the largest instance fits in 128 VGPRs without spilling).
template <bool kPaced>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
    batch_mc_kernel(const BatchArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];  // waves * kWaveBytes
    // the same in every lane of a wave, which the compiler cannot tell
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const uint32_t wbase = wave * kWaveBytes;
    unsigned long long steps = 0ull;
    // read where the launch runs, so that it fits the states there, also when
    // a graph replays it
    const bool apart = *a.apart != 0u;
    const Chunk* const chunks = apart ? a.alone : a.chunks;
    const uint32_t n_chunks = apart ? a.n_alone : a.n_chunks;
    // waves in excess of the items leave the queue alone (its counter serves one
    // at a time: 2600 of them took 30 us)
    if (blockIdx.x * (blockDim.x >> 6) + wave >= n_chunks) return;
    for (;;) {
        uint32_t ci = 0;
        if (lane == 0) ci = atomicAdd(a.queue, 1u);
        ci = __builtin_amdgcn_readfirstlane(ci);
        if (ci >= n_chunks) break;
        const Chunk ch = chunks[ci];
        const int n = (int)(__builtin_amdgcn_readfirstlane(ch.n) & ~kChunkLanes);
        run_chunk_any<kPaced>(n, a, ch, smem, wbase, lane, steps,
                              std::make_integer_sequence<int, kMaxN>{});
    }
    steps = wave_sum_u64b(steps);
    if (a.steps && lane == 0 && steps) atomicAdd(a.steps, steps);
}

}  // namespace bbe
