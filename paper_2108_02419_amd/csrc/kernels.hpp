// kernels.hpp -- kernel argument blocks and launchers shared by the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "race_common.hpp"

namespace bbe {

// Monte-Carlo over simulations sim_begin .. sim_begin + n_sims - 1 of one
// race from one state.  Passed by value (kernel arguments).
struct SimArgs {
    RaceConst rc;
    // initial state in slot order: positions ascending, equal positions by
    // competitor index; id0[k] is the competitor in slot k
    float d0[kMaxN];
    float s0[kMaxN];
    uint8_t id0[kMaxN];
    uint32_t t0;
    uint32_t sim_begin;
    uint32_t n_sims;
    uint32_t request;
    uint32_t k0, k1;  // Philox key = seed
    int stop_after;
    uint8_t* orders;            // [n_sims][n] or null
    unsigned long long* wins;   // [n], zeroed before launch, or null
    unsigned long long* steps;  // [1], zeroed before launch, or null
    RacePace pace;
};

struct PrefixArgs {
    RaceConst rc;
    float d0[kMaxN];  // slot order, as in SimArgs
    float s0[kMaxN];
    uint8_t id0[kMaxN];
    uint32_t t0;
    uint32_t request;
    uint32_t sim;
    uint32_t k0, k1;
    float target;
    uint32_t max_ticks;  // stop after this many ticks at the latest
    uint32_t* tick_out;
    float* pos_out;
    float* prev_out;
    RacePace pace;
};

int mc_block_size();
int mc_blocks_per_cu(int n, bool paced);
// the paced variants (race_kernels_paced.hip), used by the two above
int mc_blocks_per_cu_paced(int n);
hipError_t launch_race_mc_paced(const SimArgs& a, int grid, hipStream_t s);
hipError_t launch_race_mc(const SimArgs& a, int grid, hipStream_t s);
// Few simulations, a team of lanes each (team_kernels.hip), plain or paced.
bool team_mc_fits(int n, uint32_t n_sims);
hipError_t launch_team_mc(const SimArgs& a, hipStream_t s);
hipError_t launch_race_prefix(const PrefixArgs& a, hipStream_t s);
hipError_t launch_zero_u64(unsigned long long* p, int n, hipStream_t s);
// Finish-order tallies over an orders matrix [n_sims][n] (see order_kernels.hip);
// both clear their counts first.
hipError_t launch_rank_counts(const uint8_t* orders, uint32_t n_sims, int n,
                              unsigned long long* counts, hipStream_t s);
hipError_t launch_order_pmf(const uint8_t* orders, uint32_t n_sims, int n, int n_fact,
                            unsigned long long* counts, hipStream_t s);
hipError_t launch_win_probs(const unsigned long long* wins, int n_rows, int n, int stride,
                            double* probs, hipStream_t s);

}  // namespace bbe

namespace bbe {

// A start state in slot order.
struct StartState {
    float d0[kMaxN];
    float s0[kMaxN];
    uint8_t id0[kMaxN];
    uint32_t t0;
};

// One request of a batch: a race and a range of simulations of stream (seed,
// request).  Read by whole waves (uniform loads).
struct alignas(16) ReqDesc {
    RaceConst rc;
    uint32_t request;
    uint32_t sim_begin;
    uint32_t n_sims;
    int stop_after;
    RacePace pace;
};

// In-play states to generate, a record of 32-bit words each: this head, then
// elo, espan16, alpha, beta and theta of the n competitors, then gamma and tau
// (kPrefixPaced), then positions and previous steps in competitor order
// (kPrefixState; without, the race is at its start).
struct PrefixHead {
    uint32_t n;  // and the flags
    uint32_t request;
    uint32_t sim;
    uint32_t t0;
    float target;
    float L;
};
constexpr uint32_t kPrefixPaced = 0x100u, kPrefixState = 0x200u;
constexpr uint32_t kPrefixWords = sizeof(PrefixHead) / 4 + 9 * kMaxN;  // of the largest record

// A work item of the persistent kernel: simulations [first, first + count)
// of request `req` (count <= 64 * generations per chunk), or with kChunkLanes
// in `n` entries [first, first + count) of the lane table.
constexpr uint32_t kChunkLanes = 0x100u;
struct Chunk {
    uint32_t req;
    uint32_t first;
    uint32_t count;
    uint32_t n;
};

// An entry of the lane table: one simulation.
struct PackLane {
    uint32_t row;  // its request
    uint32_t sim;  // its index
};

// One launch serves the work items chunks[0 .. n_chunks) -- or, where the
// requests run apart, alone[0 .. n_alone) -- of every competitor count (chunk.n
// selects the template instance).
struct BatchArgs {
    const ReqDesc* reqs;
    const Chunk* chunks;
    const Chunk* alone;         // the items where the requests run apart
    const uint32_t* apart;      // [1]: whether they do; lies with the states
    const uint32_t* state_of;   // [n_reqs]: each request's entry of `states`
    const StartState* states;
    const PackLane* lanes;      // of the items with kChunkLanes
    uint32_t n_chunks, n_alone;
    uint32_t* queue;            // the launch's work-queue head, zeroed before launch
    unsigned long long* wins;   // [n_reqs][kMaxN], zeroed before launch
    unsigned long long* steps;  // [1] or null, zeroed before launch
    uint32_t k0, k1;
};

// paced: the items include a race with a time term of R (some gamma != 0)
hipError_t launch_batch_mc(const BatchArgs& a, int waves_per_block, int grid, bool paced,
                           hipStream_t s);
int batch_blocks_per_cu(int waves_per_block, bool paced);
// the paced variant (batch_kernels_paced.hip), used by the two above
hipError_t launch_batch_mc_paced(const BatchArgs& a, int waves_per_block, int grid,
                                 hipStream_t s);
int batch_blocks_per_cu_paced(int waves_per_block);
hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int n, hipStream_t s);
hipError_t launch_batch_probs(const unsigned long long* wins, const ReqDesc* reqs, int n_reqs,
                              double* probs, hipStream_t s);
// Record i begins at records[at[i]], or without `at` at records[kPrefixWords * i].
hipError_t launch_prefix_batch(const uint32_t* records, const uint64_t* at, int n_reqs, uint32_t k0, uint32_t k1,
                               uint32_t* tick_out, float* pos_out, float* prev_out,
                               hipStream_t s);

}  // namespace bbe
