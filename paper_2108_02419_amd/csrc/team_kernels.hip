// team_kernels.hip -- single simulations and small Monte-Carlo runs on gfx950:
// the race the bettors watch (its trace, its next state), the in-play states
// of a batch of requests (paper Section 3: the race state is the vector of
// positions, advanced tick by tick by Eq. 1), and dry-runs that are too few
// to fill the chip with a simulation a lane.
//
// A team of lanes runs one simulation, lane c for competitor c, with no order
// kept among them.  The Monte-Carlo kernels put a whole simulation in a lane
// because they have enough of them; here a tick's latency is what counts, and
// a team shortens it ninefold (the 20-competitor trace from the start, 270
// ticks: 784 us in the lane-a-race form, 90 us so, 0.33 us a tick):
//  - the competitor ahead is found by comparing with all n positions at once
//    (each lane reads them from LDS: the smallest larger one, a subtraction
//    and half a three-way minimum each, then the step of the first competitor
//    that holds it, and that only in ticks in which some lane is blocked);
//  - the draws of a tick are ceil(n/8) Philox blocks, so a team computes those
//    of G / ceil(n/8) ticks at a time, a block a lane, into an LDS table.
// One simulation has the whole wave (G = 64: its draws are made for 21 ticks
// at once at 20 competitors, and each half of the wave compares with half of
// the competitors: 134 us without the halves and the subtractions); a batch has two simulations in each wave (G =
// 32), which keeps the waves short of each other's races: in the lane-a-race
// form a wave of 64 requests with 5 to 20 competitors ran each competitor
// count's code one after the other (16384 mixed requests from the start line:
// 6.9 ms of GPU time, 0.35 ms so).
#include "bettors.hpp"
#include "kernels.hpp"
#include "race_sim.hpp"

namespace bbe {

// A lane's competitor; lanes past the last one hold a competitor that stands
// at 0 for good: ahead of nobody, and never blocked.
struct TeamLane {
    float elo = 0.0f, espan16 = 0.0f, alpha = 0.0f, beta = 0.0f, theta = -1.0f;
    float gamma = 0.0f, tau = 0.0f;
    float d = 0.0f, s = 0.0f;
};

// LDS of a team: the draw table, 8 draws a lane, and (position, step) of the
// competitors.
template <int G>
constexpr uint32_t kTeamBytes = G * 32 + kMaxN * 8;

__device__ __forceinline__ void wave_fence() {
    // the wave's LDS operations complete in order; this keeps the compiler
    // from moving them across
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lane's competitor of race rc at the state (d0, s0, id0) given in slot
// order; `pairs` is the team's table of (position, step).
__device__ __forceinline__ TeamLane team_lane(const RaceConst& rc, const RacePace& pc,
                                              const float* d0, const float* s0,
                                              const uint8_t* id0, uint32_t c, uint32_t pairs) {
    TeamLane me;
    const bool act = c < (uint32_t)rc.n;
    if (act) lds_st(pairs + 8u * id0[c], f32x2{d0[c], s0[c]});
    wave_fence();
    if (act) {
        me = {rc.elo[c],   rc.espan16[c], rc.alpha[c], rc.beta[c], rc.theta[c],
              pc.gamma[c], pc.tau[c],     0.0f,        0.0f};
        const f32x2 q = lds_ld<f32x2>(pairs + 8u * c);
        me.d = q.x;
        me.s = q.y;
    }
    wave_fence();
    return me;
}

// Ticks of every team of the wave from its tick t on, for as long as
// before(t) -- asked before each tick -- and after(crossed, cr, t) -- told
// afterwards whether somebody reached the line, whether this lane's
// competitor did, and the next tick -- both hold for the team (they give the
// same answer in all its lanes).  A competitor at NaN has left the race.  A
// competitor that reaches the line keeps its position of before the tick.
// J >= n (a multiple of 4): the competitors looked at.  A team that has the
// whole wave (G = 64) is there twice, lanes 32 + c as lanes c, and each half
// looks at half of the competitors.
template <int G, int J, class Before, class After>
__device__ __forceinline__ void team_run(TeamLane& me, uint32_t c, uint32_t n, uint32_t draws,
                                         uint32_t pairs, float L, uint32_t t, uint32_t sim,
                                         uint32_t request, uint32_t k0, uint32_t k1, bool run,
                                         Before&& before, After&& after) {
    constexpr uint32_t kBlocks = (J + 7) / 8;  // of the largest team of the wave
    constexpr uint32_t kAhead = G / kBlocks;   // ticks whose draws are made at once
    const uint32_t nb = (n + 7u) / 8u;
    const uint32_t my_tick = c / nb, my_block = c - my_tick * nb;
    constexpr int kHalves = G == 64 ? 2 : 1, kRows = J / 2 / kHalves;
    const uint32_t me_at = kHalves == 2 ? c & 31u : c;
    const uint32_t look = pairs + (kHalves == 2 ? (c >> 5) * (16u * kRows) : 0u);
    const uint32_t place = draws + 4u * min(me_at, n - 1u);
    const uint64_t team = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1) << (__lane_id() & ~(G - 1));
    uint32_t i = kAhead;
    for (;;) {
        run = run && before(t);
        if (!__builtin_amdgcn_ballot_w64(run)) break;
        if (i == kAhead) {
            i = 0;
            const U4 w = philox4x32_10(t + my_tick, sim, request, my_block, k0, k1);
            if (my_tick < kAhead) {
                lds_st(draws + 32u * c,
                       f32x4{draw_hi(w.x), draw_lo(w.x), draw_hi(w.y), draw_lo(w.y)});
                lds_st(draws + 32u * c + 16u,
                       f32x4{draw_hi(w.z), draw_lo(w.z), draw_hi(w.w), draw_lo(w.w)});
            }
        }
        if (c < (uint32_t)J) lds_st(pairs + 8u * c, f32x2{me.d, me.s});
        wave_fence();
        f32x4 q[kRows];
#pragma unroll
        for (int j = 0; j < kRows; ++j) q[j] = lds_ld<f32x4>(look + 16u * j);
        const float u = lds_ld<float>(place + 32u * nb * i);
        wave_fence();
        float R = me.alpha + me.beta * me.d;
        R = R + me.gamma * fminf((float)t, me.tau);
        float f = me.elo + me.espan16 * u;
        // the smallest position ahead, from the distances between the bits
        // (positions are >= 0: ordered like their bits; nobody ahead, and
        // oneself, wrap to 2^31 and more)
        const uint32_t past = __float_as_uint(me.d) + 1u;
        uint32_t near = ~0u;
#pragma unroll
        for (int j = 0; j < kRows; ++j)
            near = min(near, min(__float_as_uint(q[j].x) - past, __float_as_uint(q[j].z) - past));
        if constexpr (kHalves == 2) {
            const auto h = __builtin_amdgcn_permlane32_swap(near, near, false, false);
            near = min(h[0], h[1]);
        }
        const float nd = __uint_as_float(near + past);
        const bool blocked = (int)near >= 0 && nd - me.d <= me.theta;
        if (__builtin_amdgcn_ballot_w64(blocked)) {
            float ns = -1.0f;  // step of the lowest index among equal positions
#pragma unroll
            for (int j = kRows - 1; j >= 0; --j) {
                ns = q[j].z == nd ? q[j].w : ns;
                ns = q[j].x == nd ? q[j].y : ns;
            }
            if constexpr (kHalves == 2) {
                const uint32_t v = __float_as_uint(ns);
                const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
                ns = __uint_as_float((int)h[0] >= 0 ? h[0] : h[1]);
            }
            const float s_min =
                __uint_as_float(min(__float_as_uint(me.s), __float_as_uint(ns)));
            f = blocked ? s_min : f;
        }
        const float S = R * f;
        const float dn = me.d + S;
        const bool cr = dn >= L;
        const bool crossed = (__builtin_amdgcn_ballot_w64(cr) & team) != 0;
        if (run) {
            me.d = cr ? me.d : dn;
            me.s = S;
            t += 1;
            run = after(crossed, cr, t);
        }
        i += 1;
    }
}

// Instance of team_run for the largest n of the wave (at most G).
template <int G, class Before, class After>
__device__ __forceinline__ void team_run_any(uint32_t n_max, TeamLane& me, uint32_t c,
                                             uint32_t n, uint32_t draws, uint32_t pairs, float L,
                                             uint32_t t, uint32_t sim, uint32_t request,
                                             uint32_t k0, uint32_t k1, bool run, Before&& before,
                                             After&& after) {
    switch ((n_max + 3u) / 4u) {
#define BBE_CASE(m)                                                                            \
    case m:                                                                                    \
        if constexpr (4 * m <= G)                                                              \
            team_run<G, 4 * m>(me, c, n, draws, pairs, L, t, sim, request, k0, k1, run,        \
                               before, after);                                                 \
        break;
        BBE_CASE(1) BBE_CASE(2) BBE_CASE(3) BBE_CASE(4) BBE_CASE(5)
#undef BBE_CASE
        default:
            break;
    }
}

// One simulation until its leader reaches the target.
__global__ void __launch_bounds__(64) race_prefix_kernel(const PrefixArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[kTeamBytes<64>];
    const uint32_t c = threadIdx.x, n = (uint32_t)a.rc.n;
    const uint32_t draws = lds_addr(smem), pairs = draws + 64 * 32;
    TeamLane me = team_lane(a.rc, a.pace, a.d0, a.s0, a.id0, c & 31u, pairs);
    uint32_t t_end = a.t0;
    bool ok = true;
    team_run_any<64>(
        n, me, c, n, draws, pairs, a.rc.L, a.t0, a.sim, a.request, a.k0, a.k1, true,
        [&](uint32_t t) {
            if (__builtin_amdgcn_ballot_w64(me.d >= a.target)) return false;
            if (t - a.t0 >= a.max_ticks) return false;
            if (t - a.t0 >= kTickLimit) {
                ok = false;
                return false;
            }
            return true;
        },
        [&](bool crossed, bool, uint32_t t) {
            t_end = t;
            ok = !crossed;
            return !crossed;
        });
    if (c == 0) *a.tick_out = ok ? t_end : 0xFFFFFFFFu;
    if (c < n) {
        a.pos_out[c] = me.d;
        a.prev_out[c] = me.s;
    }
}

// Positions of one simulation, a row per tick.
__global__ void __launch_bounds__(64) race_trace_kernel(const TraceArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[kTeamBytes<64>];
    const uint32_t c = threadIdx.x, n = (uint32_t)a.rc.n;
    const uint32_t draws = lds_addr(smem), pairs = draws + 64 * 32;
    TeamLane me = team_lane(a.rc, a.pace, a.d0, a.s0, a.id0, c & 31u, pairs);
    if (c < n) a.trace[c] = me.d;
    uint32_t rows = 1;
    // at most max_rows - 1 <= 2^20 ticks
    team_run_any<64>(
        n, me, c, n, draws, pairs, a.rc.L, a.t0, a.sim, a.request, a.k0, a.k1, true,
        [&](uint32_t) { return rows < a.max_rows; },
        [&](bool crossed, bool, uint32_t) {
            if (crossed) return false;
            if (c < n) a.trace[(size_t)rows * n + c] = me.d;
            rows += 1;
            return true;
        });
    if (c == 0) *a.rows_out = rows;
}

// In-play states for a batch: team i advances the simulation of record i until
// its leader reaches the target.
__global__ void __launch_bounds__(64)
    prefix_batch_kernel(const uint32_t* __restrict__ records, const uint64_t* __restrict__ at,
                        int n_reqs, uint32_t k0, uint32_t k1, uint32_t* __restrict__ tick_out,
                        float* __restrict__ pos_out, float* __restrict__ prev_out) {
    constexpr int G = 32;
    __shared__ __attribute__((aligned(16))) char smem[2 * kTeamBytes<G>];
    const uint32_t half = threadIdx.x / G, c = threadIdx.x % G;
    const uint32_t draws = lds_addr(smem) + half * kTeamBytes<G>, pairs = draws + G * 32;
    const int i = 2 * (int)blockIdx.x + (int)half;
    const bool have = i < n_reqs;
    // an odd batch's last half-wave idles through its neighbour's race
    const int mine = have ? i : n_reqs - 1;
    const uint32_t* w = records + (at ? (size_t)at[mine] : (size_t)mine * kPrefixWords);
    PrefixHead rq;
    __builtin_memcpy(&rq, w, sizeof rq);
    w += sizeof rq / 4;
    const uint32_t n = rq.n & 0xFFu;
    const uint32_t n_max =
        max((uint32_t)__builtin_amdgcn_readlane(n, 0), (uint32_t)__builtin_amdgcn_readlane(n, G));
    TeamLane me;
    if (c < n) {
        const float* v = reinterpret_cast<const float*>(w) + c;
        me = {v[0], v[n], v[2 * n], v[3 * n], v[4 * n], 0.0f, 0.0f, 0.0f, 0.0f};
        v += 5 * n;
        if (rq.n & kPrefixPaced) {
            me.gamma = v[0];
            me.tau = v[n];
            v += 2 * n;
        }
        if (rq.n & kPrefixState) {
            me.d = v[0];
            me.s = v[n];
        }
    }
    const uint64_t team = 0xFFFFFFFFull << (half * G);
    const float target = rq.target;
    const uint32_t t0 = rq.t0;
    uint32_t t_end = t0;
    bool ok = true;
    team_run_any<G>(
        n_max, me, c, n, draws, pairs, rq.L, t0, rq.sim, rq.request, k0, k1, have,
        [&](uint32_t t) {
            if (__builtin_amdgcn_ballot_w64(me.d >= target) & team) return false;
            if (t - t0 >= kTickLimit) {
                ok = false;
                return false;
            }
            return true;
        },
        [&](bool crossed, bool, uint32_t t) {
            t_end = t;
            ok = !crossed;
            return !crossed;
        });
    if (!have) return;
    if (c == 0) tick_out[i] = ok ? t_end : 0xFFFFFFFFu;
    if (c < (uint32_t)kMaxN) {
        pos_out[(size_t)i * kMaxN + c] = c < n ? me.d : 0.0f;
        prev_out[(size_t)i * kMaxN + c] = c < n ? me.s : 0.0f;
    }
}

// Monte-Carlo dry-runs, a team each (see launch_team_mc for when): finish
// orders, win counts and competitor-steps as race_mc_kernel gives them.
constexpr int kTeamMcBlock = 256;

template <int G>
__global__ void __launch_bounds__(kTeamMcBlock) team_mc_kernel(const SimArgs a) {
    constexpr int kTeams = kTeamMcBlock / G;
    __shared__ __attribute__((aligned(16))) char smem[kTeams * kTeamBytes<G>];
    __shared__ uint32_t s_wins[kMaxN];
    __shared__ unsigned long long s_steps;
    const uint32_t c = threadIdx.x % G, n = (uint32_t)a.rc.n;
    const uint32_t draws = lds_addr(smem) + (threadIdx.x / G) * kTeamBytes<G>;
    const uint32_t pairs = draws + G * 32;
    if (threadIdx.x < kMaxN) s_wins[threadIdx.x] = 0u;
    if (threadIdx.x == 0) s_steps = 0ull;
    __syncthreads();
    const uint32_t base = __lane_id() & ~(uint32_t)(G - 1);
    const uint64_t team = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1) << base;
    unsigned long long steps = 0ull;
    // a wave's teams take neighbouring simulations and go on together
    for (uint64_t first = ((uint64_t)blockIdx.x * kTeamMcBlock + (threadIdx.x & ~63u)) / G;
         first < a.n_sims; first += (uint64_t)gridDim.x * kTeams) {
        const uint64_t j = first + (threadIdx.x & 63u) / G;
        const bool have = j < a.n_sims;
        uint8_t* row = a.orders ? a.orders + (have ? j : 0) * n : nullptr;
        TeamLane me = team_lane(a.rc, a.pace, a.d0, a.s0, a.id0, c, pairs);
        uint32_t nfin = 0, ran = 0;
        team_run_any<G>(
            n, me, c, n, draws, pairs, a.rc.L, a.t0, a.sim_begin + (uint32_t)j, a.request, a.k0,
            a.k1, have, [](uint32_t) { return true; },
            [&](bool crossed, bool cr, uint32_t t) {
                if (crossed) {
                    // finishers of one tick by crossing fraction, then index
                    const uint64_t who = __builtin_amdgcn_ballot_w64(cr) & team;
                    uint32_t rank = nfin;
                    if (who & (who - 1)) {
                        const float f = (a.rc.L - me.d) / me.s;
                        if (cr) lds_st(pairs + 8u * c, f);
                        wave_fence();
                        if (cr)
                            for (uint64_t m = who; m; m &= m - 1) {
                                const uint32_t o = (uint32_t)__builtin_ctzll(m) - base;
                                const float fo = lds_ld<float>(pairs + 8u * o);
                                rank += fo < f || (fo == f && o < c) ? 1u : 0u;
                            }
                        wave_fence();
                    }
                    if (cr) {
                        if (rank == 0) atomicAdd(&s_wins[c], 1u);
                        if (row) row[rank] = (uint8_t)c;
                        ran = t - a.t0;
                        me.d = parked();
                    }
                    nfin += (uint32_t)__popcll(who);
                }
                if (nfin < (uint32_t)a.stop_after && t - a.t0 < kTickLimit) return true;
                if (c < n && me.d == me.d) ran = t - a.t0;
                if (row && c >= nfin && c < n) row[c] = 0xFF;
                return false;
            });
        steps += have ? ran : 0u;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) steps += __shfl_xor(steps, off, 64);
    if ((threadIdx.x & 63) == 0 && steps) atomicAdd(&s_steps, steps);
    __syncthreads();
    if (a.wins && threadIdx.x < n && s_wins[threadIdx.x])
        atomicAdd(&a.wins[threadIdx.x], (unsigned long long)s_wins[threadIdx.x]);
    if (a.steps && threadIdx.x == 0 && s_steps) atomicAdd(a.steps, s_steps);
}

// ---------------------------------------------------------------- launchers

hipError_t launch_race_prefix(const PrefixArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(race_prefix_kernel, dim3(1), dim3(64), 0, s, a);
    return hipGetLastError();
}

// Whether n_sims dry-runs of n competitors end sooner with a team each than
// with a lane each.  A lane each takes as long as one simulation does in a
// lane, however few there are (until 4 waves a SIMD are full); teams take a
// fraction of that, but of every wave they fill, so the line lies where their
// waves begin to queue: at so many simulations per competitor for teams of 8,
// 16 and 32 lanes.  Measured on both sides, full orders, us (team / lane):
//   n = 2   1000: 116 / 139     8192: 118 / 139     16384: 123 / 139
//   n = 3   1000: 120 / 181    12288: 125 / 181     24576: 139 / 181
//   n = 4   1000: 120 / 220    16384: 128 / 220     32768: 155 / 220
//   n = 5   1000: 128 / 261    30720: 176 / 261     40960: 200 / 261
//   n = 8  49152: 237 / 362    65536: 298 / 362
//   n = 13 10400: 219 / 601    31200: 443 / 601     41600: 577 / 601
//   n = 17 19125: 607 / 805    25500: 760 / 805
//   n = 20  7500: 299 / 948    22500: 676 / 948     30000: 884 / 948
// The lead is least where a run is short (to the winner with a tenth of the track
// to go, n = 8, 65536: 69 / 65).  One competitor needs no look at the others: a
// lane each, 80 against 105.
bool team_mc_fits(int n, uint32_t n_sims) {
    if (n < 2) return false;
    const uint32_t per = n <= 8 ? 8192u : n <= 16 ? 3200u : 1500u;
    return n_sims <= per * (uint32_t)n;
}

hipError_t launch_team_mc(const SimArgs& a, hipStream_t s) {
    const int n = a.rc.n;
    const uint32_t lanes = n <= 8 ? 8 : n <= 16 ? 16 : 32;
    const dim3 grid((unsigned)(((uint64_t)a.n_sims * lanes + kTeamMcBlock - 1) / kTeamMcBlock));
    if (n <= 8)
        hipLaunchKernelGGL(team_mc_kernel<8>, grid, dim3(kTeamMcBlock), 0, s, a);
    else if (n <= 16)
        hipLaunchKernelGGL(team_mc_kernel<16>, grid, dim3(kTeamMcBlock), 0, s, a);
    else
        hipLaunchKernelGGL(team_mc_kernel<32>, grid, dim3(kTeamMcBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_race_trace(const TraceArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(race_trace_kernel, dim3(1), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_prefix_batch(const uint32_t* records, const uint64_t* at, int n_reqs,
                               uint32_t k0, uint32_t k1, uint32_t* tick_out, float* pos_out,
                               float* prev_out, hipStream_t s) {
    if (n_reqs <= 0) return hipSuccess;
    hipLaunchKernelGGL(prefix_batch_kernel, dim3((unsigned)(((long)n_reqs + 1) / 2)), dim3(64), 0,
                       s, records, at, n_reqs, k0, k1, tick_out, pos_out, prev_out);
    return hipGetLastError();
}

}  // namespace bbe
