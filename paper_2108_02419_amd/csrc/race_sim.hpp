// race_sim.hpp -- one simulated race per lane, 64 lanes in lockstep
// (paper Section 3, Eq. 1).
//
// Layout.  A lane keeps its competitors in N register "slots" sorted by
// position (ascending; finished competitors are parked at the top with a
// NaN position).  Slot k holds the position d[k], the LDS byte offset
// rec[k] of its competitor's parameter record (pbase + 16 * competitor
// index; it also locates the competitor's draw) and the previous step s[k].
// Slots are ordered by the 64-bit key (bits(d) << 32) | rec: non-negative
// floats, +inf and the parking NaN order like their bit patterns, and rec
// grows with the competitor index, so this is (position, index) order.  The
// competitor ahead of slot k is then the first slot above it with a larger
// position -- slot k+1 unless positions are equal -- and the query of Eq. 1
// costs O(1) per competitor instead of a scan over all pairs.
//
// One tick (all 64 lanes at the same absolute tick t):
//   1. draws in competitor order: Philox4x32-10(key = seed,
//      ctr = (t, sim, request, b)) for blocks b = 0 .. ceil(N/8)-1;
//      competitor c takes word (c>>1)&3 of block c>>3, its high half for
//      even c and its low half for odd c, as the integer k (u = k * 2^-16);
//      the draws go to the lane's column of an LDS table and each slot
//      reads the draw of its own competitor;
//   2. competitor ahead: the running competitor with the smallest position
//      greater than d_c (lowest index among equal positions); gap =
//      fl(d_ahead - d_c), +inf if nobody is ahead;
//   3. Eq. 1: R = alpha + beta*d (+ gamma*min(t, tau) in the paced
//      variants); free: S = R*(elo + espan*u); blocked (gap <= theta):
//      S = R*min(s_c, s_ahead);
//   4. synchronous update d += S, s = S of the running competitors; a
//      competitor whose new position reaches L crosses the line;
//   5. this tick's finishers are ranked after the earlier ones, among
//      themselves by the fraction fl((L - d_old)/S), then by index, and are
//      parked (position NaN: every comparison with it is false, so a parked
//      slot never crosses again and is never "ahead" of anyone);
//   6. compare-exchange passes, alternately upward and downward, restore the
//      slot order.
//
// slots_tick does this in full.  The Monte-Carlo kernels use it only where two
// positions are equal, and slots_tick_plain (below) everywhere else.
#pragma once

#include "race_common.hpp"

#include <type_traits>

namespace bbe {

template <int N>
struct Slots {
    float d[N];
    uint32_t rec[N];
    float s[N];
};

// Order key of a slot.
__device__ __forceinline__ uint64_t slot_key(float d, uint32_t rec) {
    return ((uint64_t)__float_as_uint(d) << 32) | rec;
}

// LDS by address.  The kernels' tables are one array each, addressed by byte
// offsets that sit in registers; through a pointer to the array every access
// paid an add of its base.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <class T>
using LdsPtr = __attribute__((address_space(3))) T*;

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(LdsPtr<const void>)p;
}
template <class T>
__device__ __forceinline__ T lds_ld(uint32_t addr) {
    return *(LdsPtr<const T>)(uintptr_t)addr;
}
template <class T>
__device__ __forceinline__ void lds_st(uint32_t addr, T v) {
    *(LdsPtr<T>)(uintptr_t)addr = v;
}

// This lane's index, opaque to the compiler: what depends on it is computed
// where it is used and holds no register -- or spill slot -- across a tick.
__device__ __forceinline__ uint32_t lane_here() {
    uint32_t lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

constexpr uint32_t kNoRow = 0xFFFFFFFFu;  // no finish order wanted

// The parking position of finished competitors (a quiet NaN whose bit
// pattern exceeds that of +inf).
__device__ __forceinline__ float parked() {
    return __uint_as_float(0x7FC00000u);
}

// How a tick adds the time term gamma*min(t, tau) of R: not at all (gamma = 0
// everywhere), or from a table: all lanes of the wave are at the same tick, so
// lane c forms competitor c's term once per tick into its record and every
// slot adds it.
enum Pace : int { kPaceOff = 0, kPaceTable = 1 };

// Parameter records: competitor c's (elo, espan16, alpha, beta) at
// pbase + 16*c and (theta, term, tau, gamma) at the same distance from the
// second half of the table; tau and gamma are written (by the same lane,
// afterwards) by write_pace, the current tick's term by write_pace_terms.
// In two halves
// because the slots of a wave read 64 records at once: at 16 bytes apart two
// of up to 16 competitors never share a bank, at 32 bytes competitors eight
// apart did (bank conflicts 28 -> 13% of the cycles at 20 competitors).
constexpr uint32_t kRecSize = 16;
template <int N>
constexpr uint32_t kRecHalf = kRecSize * N;

// Writes the parameter records of a race.
template <int N>
__device__ __forceinline__ void write_params(uint32_t pbase, const RaceConst& rc,
                                            int lane) {
    if (lane < N) {
        const uint32_t rec = pbase + kRecSize * lane;
        lds_st(rec, f32x4{rc.elo[lane], rc.espan16[lane], rc.alpha[lane], rc.beta[lane]});
        lds_st(rec + kRecHalf<N>, f32x4{rc.theta[lane], 0.0f, 0.0f, 0.0f});
    }
}

template <int N>
__device__ __forceinline__ void write_pace(uint32_t pbase, const RacePace& pc,
                                          int lane) {
    if (lane < N) {
        const uint32_t rec = pbase + kRecSize * lane + kRecHalf<N>;
        lds_st(rec + 8u, pc.tau[lane]);
        lds_st(rec + 12u, pc.gamma[lane]);
    }
}

// Loads an initial state already in slot order (positions ascending, equal
// positions by competitor index); `pbase` locates the parameter records.
template <int N>
__device__ __forceinline__ void slots_reset(Slots<N>& sl, const float* __restrict__ d0,
                                            const float* __restrict__ s0,
                                            const uint8_t* __restrict__ id0, uint32_t pbase) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        sl.d[k] = d0[k];
        sl.rec[k] = pbase + kRecSize * id0[k];
        sl.s[k] = s0[k];
    }
}

// This tick's time term of competitor c, formed by lane c (t is the same in
// every lane) into its record for the wave's slots to add.
template <int N>
__device__ __forceinline__ void write_pace_terms(uint32_t pbase, uint32_t t) {
    const uint32_t lane = __lane_id();
    if (lane < (uint32_t)N) {
        const uint32_t r = pbase + kRecSize * lane + kRecHalf<N>;
        const f32x2 tg = lds_ld<f32x2>(r + 8u);  // (tau, gamma)
        lds_st<float>(r + 4u, tg.y * fminf((float)t, tg.x));
    }
    // the wave's LDS operations complete in order; keep the compiler
    // from moving the slots' reads above this store
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Step 1: writes this tick's draws of a lane's competitors into its column.
template <int N>
__device__ __forceinline__ void write_draws(uint32_t ucol, uint32_t t, uint32_t sim,
                                            uint32_t request, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int b = 0; b < (N + 7) / 8; ++b) {
        const U4 w = philox4x32_10(t, sim, request, (uint32_t)b, k0, k1);
        const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = 8 * b + 2 * j;
            if (c < N) lds_st<float>(ucol + c * 256, draw_hi(words[j]));
            if (c + 1 < N) lds_st<float>(ucol + (c + 1) * 256, draw_lo(words[j]));
        }
    }
}

// Steps 1-4 for one lane.  `ucol` is the byte offset of this lane's column
// of the draw table (competitor c's draw at ucol + 256*c), `pbase` that of
// the parameter records.  Returns the bit mask of slots that crossed the
// line (their position still holds the start-of-tick value; their s holds
// the step S that took them over).  kPace selects how the time term of R
// is added (with gamma = 0 it adds +0, so every mode agrees on unpaced
// races).  A parked slot's step changes nothing: it stays parked and is never
// ahead of anyone.
template <int N, Pace kPace = kPaceOff>
__device__ __forceinline__ uint32_t slots_tick(Slots<N>& sl, uint32_t ucol,
                                               uint32_t pbase, float L, uint32_t t,
                                               uint32_t sim, uint32_t request, uint32_t k0,
                                               uint32_t k1) {
    if constexpr (kPace == kPaceTable) {
        write_pace_terms<N>(pbase, t);
    }
    // 1. draws, competitor order, into this lane's column
    write_draws<N>(ucol, t, sim, request, k0, k1);

    // 2.-4. Slots from the top down.  Slots are in (position, index) order,
    //    so the competitor ahead of slot k is the first slot above it with a
    //    larger position: slot k+1, or -- where positions are equal -- the
    //    one found for slot k+1, carried down in (nd, ns).  The start-of-tick
    //    position and step of slot k+1 are kept in (d_up, s_up) because the
    //    update overwrites the slot (synchronous update).  The draw of
    //    competitor c sits at ucol + 256*c = ubias + 16*rec; each slot's draw
    //    and parameter record are read from LDS kPf slots ahead of use.
    const uint32_t ubias = ucol - 16u * pbase;
    constexpr int kPf = 4;
    float pu[N], pth[N], pga[N];
    f32x4 pp[N];
#pragma unroll
    for (int k = N - 1; k >= 0 && k >= N - kPf; --k) {
        const uint32_t rec = sl.rec[k];
        pu[k] = lds_ld<float>(ubias + (rec << 4));
        pp[k] = lds_ld<f32x4>(rec);
        if constexpr (kPace == kPaceTable) {
            const f32x2 q = lds_ld<f32x2>(rec + kRecHalf<N>);
            pth[k] = q.x;
            pga[k] = q.y;  // the term itself
        } else {
            pth[k] = lds_ld<float>(rec + kRecHalf<N>);
        }
    }
    float nd = __builtin_inff(), ns = 0.0f;
    float d_up = __builtin_inff(), s_up = 0.0f;
    uint32_t cross = 0;
#pragma unroll
    for (int k = N - 1; k >= 0; --k) {
        if (k - kPf >= 0) {
            const uint32_t rec = sl.rec[k - kPf];
            pu[k - kPf] = lds_ld<float>(ubias + (rec << 4));
            pp[k - kPf] = lds_ld<f32x4>(rec);
            if constexpr (kPace == kPaceTable) {
                const f32x2 q = lds_ld<f32x2>(rec + kRecHalf<N>);
                pth[k - kPf] = q.x;
                pga[k - kPf] = q.y;
            } else {
                pth[k - kPf] = lds_ld<float>(rec + kRecHalf<N>);
            }
        }
        const float d = sl.d[k];
        const float s = sl.s[k];
        const bool gt = d_up > d;  // false next to a parked (NaN) slot
        nd = gt ? d_up : nd;
        ns = gt ? s_up : ns;
        // Eq. 1
        const f32x4 p = pp[k];
        float R = p.z + p.w * d;
        if constexpr (kPace == kPaceTable) R = R + pga[k];
        float x = p.x + p.y * pu[k];
        // min of two positive steps (ns = 0 only when nobody is ahead)
        float s_min = __uint_as_float(min(__float_as_uint(s), __float_as_uint(ns)));
        float gap = nd - d;  // +inf when nobody is ahead
        // R*s_min when blocked, R*x when free (one product of the selected
        // factor rounds exactly as the product taken in that branch)
        float S = R * ((gap <= pth[k]) ? s_min : x);
        // synchronous update; a parked slot computes NaN and stays parked
        float dn = d + S;
        bool cr = dn >= L;
        cross = cross + cross + (cr ? 1u : 0u);  // slot k lands on bit k
        sl.d[k] = cr ? d : dn;
        sl.s[k] = S;
        d_up = d;
        s_up = s;
    }
    return cross;
}

// Step 5: ranks this tick's finishers (slot mask `cross`) after the `nfin`
// earlier ones, records them, and parks every crossing slot (position NaN);
// returns the number ranked.  `rank` is false in lanes whose simulation has
// already ended: their finishers are parked but not recorded.  In one pass
// over the crossing slots, each finisher is compacted -- entry j (the j-th
// set bit of `cross`) holds its competitor index in the lane's column of a
// byte table, at icol + 64*j, and, when there are several, its crossing
// fraction in the lane's (already consumed) column of the draw table, at
// ucol + 256*j -- and its slot is parked.  The entries are then picked in
// (fraction, index) order by a selection over those c entries, so the work
// grows with c^2 for the few finishers of a tick rather than with c*N.
template <int N, class Win>
__device__ __forceinline__ int slots_rank_park(Slots<N>& sl, uint32_t cross, bool rank, float L,
                                               uint32_t ucol, uint32_t icol, uint32_t pbase,
                                               int nfin, const Win& win, uint32_t row) {
    const int c = __builtin_popcount(cross);
#pragma unroll
    for (int k = 0; k < N; ++k)
        if ((cross >> k) & 1u) {
            if (rank) {
                const uint32_t j = __builtin_popcount(cross & ((1u << k) - 1u));
                lds_st<uint8_t>(icol + 64u * j, (uint8_t)((sl.rec[k] - pbase) >> 4));
                // a lone finisher needs no fraction
                if (c > 1) lds_st<float>(ucol + 256u * j, (L - sl.d[k]) / sl.s[k]);
            }
            sl.d[k] = parked();
        }
    if (!rank) return 0;
    uint32_t used = 0u;
    for (int r = 0; r < c; ++r) {
        int bj = -1;
        float bf = 0.0f;
        uint32_t bid = 0u;
        for (int j = 0; j < c; ++j) {
            const float f = lds_ld<float>(ucol + 256u * j);
            const uint32_t id = lds_ld<uint8_t>(icol + 64u * j);
            const bool better =
                !((used >> j) & 1u) && ((bj < 0) || (f < bf) || (f == bf && id < bid));
            bj = better ? j : bj;
            bf = better ? f : bf;
            bid = better ? id : bid;
        }
        used |= 1u << bj;  // c - r > 0 entries are unused, so bj >= 0
        const int rr = nfin + r;
        if (rr == 0) win(bid);
        if (row != kNoRow) lds_st<uint8_t>(row + rr, (uint8_t)bid);
    }
    return c;
}

// Step 6: compare-exchange of slots k and k+1: three v_swap_b32 under the
// execution mask of the lanes that need the exchange, skipped when none
// does (the first pass of a tick exchanges most pairs in some lane, later
// passes few).
__device__ __forceinline__ void vswap(float& a, float& b) {
    asm volatile("v_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void vswap(uint32_t& a, uint32_t& b) {
    asm volatile("v_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}

template <int N>
__device__ __forceinline__ void slots_cx(Slots<N>& sl, int k) {
    if (slot_key(sl.d[k], sl.rec[k]) > slot_key(sl.d[k + 1], sl.rec[k + 1])) {
        vswap(sl.d[k], sl.d[k + 1]);
        vswap(sl.rec[k], sl.rec[k + 1]);
        vswap(sl.s[k], sl.s[k + 1]);
    }
}

// One upward pass that also re-exchanges the pair below after each step
// (k = 0 .. N-2: pairs k, then k-1), so a slot passed by two others moves
// down two places in one pass.  A tick's overtakes then need one such pass
// in most ticks where plain up/down passes need two: by a CPU replay of
// the 20-competitor workload, 1.24 passes and 22 order checks per tick
// instead of 2.22 and 40, for the same number of compare-exchanges.
// Checks every pair once the pass has left it.
template <int N>
__device__ __forceinline__ bool slots_pass_up2(Slots<N>& sl) {
    bool bad = false;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        slots_cx<N>(sl, k);
        if (k >= 1) slots_cx<N>(sl, k - 1);
        if (k >= 2)
            bad |= slot_key(sl.d[k - 2], sl.rec[k - 2]) > slot_key(sl.d[k - 1], sl.rec[k - 1]);
    }
    if constexpr (N >= 3)
        bad |= slot_key(sl.d[N - 3], sl.rec[N - 3]) > slot_key(sl.d[N - 2], sl.rec[N - 2]);
    if constexpr (N >= 2)
        bad |= slot_key(sl.d[N - 2], sl.rec[N - 2]) > slot_key(sl.d[N - 1], sl.rec[N - 1]);
    return bad;
}

// One downward pass (k = N-2 .. 0; carries a slot down any distance).
template <int N>
__device__ __forceinline__ bool slots_pass_down(Slots<N>& sl) {
    bool bad = false;
#pragma unroll
    for (int k = N - 2; k >= 0; --k) {
        slots_cx<N>(sl, k);
        if (k + 2 <= N - 1)
            bad |= slot_key(sl.d[k + 1], sl.rec[k + 1]) > slot_key(sl.d[k + 2], sl.rec[k + 2]);
    }
    return bad;
}

// Step 6 in full: alternate passes until every active lane of the wave is
// in order (a tick's overtakes need one pass in most lanes, two where a
// slot moves down by more than two places).
template <int N>
__device__ __forceinline__ void slots_restore(Slots<N>& sl) {
    for (;;) {
        if (!__builtin_amdgcn_ballot_w64(slots_pass_up2<N>(sl))) break;
        if (!__builtin_amdgcn_ballot_w64(slots_pass_down<N>(sl))) break;
    }
}

// ---------------------------------------------------------------------------
// Plain ticks: no two running competitors of a lane share a position.  Nearly
// every tick of a wave is plain (equal positions: the start line, and a few
// ticks in ten thousand after it), and needs much less than slots_tick: the
// competitor ahead of slot k is slot k+1 itself, and float compares order the
// slots (no compare with a parked slot's NaN holds, which leaves the parked
// slots at the top and whoever leads unblocked).  Ticks that are not plain
// take slots_tick and its passes.
//
// At 20 competitors a plain tick's straight-line block has 308 vector
// instructions against 466 of slots_tick, and its sort 19 compares and what
// has to move against 42 compares and 22 checks.  The kernels are bound by
// vector issue (98% busy over the uneven batch), so that is the gain: 10^6
// simulations of 20 competitors from the start 7.54 -> 5.93 ms, 4096 uneven
// in-play requests 19.95 -> 16.4 ms.  A race whose competitors stay tied for
// good pays for both: 13% more than before.
// ---------------------------------------------------------------------------

struct StepBounds {
    float step_cap, reach2, reach8;  // as in RaceConst
};

// Ticks (8, 2 or 0) in which no competitor of any lane can reach the line.
// A step is at most R times the largest of step_cap and the steps of the tick
// before, so the leader's position plus that step times r + r^2 + ... bounds
// every position of the ticks to come.  A parked slot (NaN) gives 0.
template <int N>
__device__ __forceinline__ int open_ticks(const Slots<N>& sl, float L, const StepBounds& sb) {
    uint32_t m = __float_as_uint(sb.step_cap);
#pragma unroll
    for (int k = 0; k < N; ++k) m = max(m, __float_as_uint(sl.s[k]));
    const float step = __uint_as_float(m);
    const float line = L * (1.0f - 0x1p-18f);  // room for the roundings of the sums
    const float top = sl.d[N - 1];
    if (!__builtin_amdgcn_ballot_w64(!(top + step * sb.reach8 < line))) return 8;
    if (!__builtin_amdgcn_ballot_w64(!(top + step * sb.reach2 < line))) return 2;
    return 0;
}

// Distance from slot k to slot k+1 of the A lowest slots (NaN below a parked
// slot, +inf for the top one) and whether some lane of the wave has two equal
// positions.
template <int N, int A>
__device__ __forceinline__ bool slots_gaps(const Slots<N>& sl, float (&gap)[N]) {
    uint32_t least = 0x7F800000u;
#pragma unroll
    for (int k = 0; k < A - 1; ++k) {
        gap[k] = sl.d[k + 1] - sl.d[k];
        least = min(least, __float_as_uint(gap[k]));  // gaps are >= 0: ordered like their bits
    }
    gap[A - 1] = __builtin_inff();
    return __builtin_amdgcn_ballot_w64(least == 0u) != 0;
}

// Whether some lane of the wave has two equal positions (parked slots, whose
// NaN equals nothing, apart).
template <int N>
__device__ __forceinline__ bool slots_tied(const Slots<N>& sl) {
    bool tie = false;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) tie |= sl.d[k] == sl.d[k + 1];
    return __builtin_amdgcn_ballot_w64(tie) != 0;
}

// Keeps the compiler from carrying one loop's choice of registers for the
// slots into another (the 64-bit compares of the other ticks want position
// and record in a register pair; with one choice for all, the loop of the
// plain ticks began with 60 moves).
template <int N>
__device__ __forceinline__ void slots_opaque(Slots<N>& sl) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        float d, s;
        uint32_t rec;
        asm volatile("v_mov_b32 %0, %3\n\tv_mov_b32 %1, %4\n\tv_mov_b32 %2, %5"
                     : "=&v"(d), "=&v"(rec), "=&v"(s)
                     : "v"(sl.d[k]), "v"(sl.rec[k]), "v"(sl.s[k]));
        sl.d[k] = d;
        sl.rec[k] = rec;
        sl.s[k] = s;
    }
}

// Moves slot K down past the up to three slots below it with larger
// positions, in every lane, slots 0 .. K-1 being in order: afterwards slots
// 0 .. K are, but in the lanes of `deep`, where slot K moved three places and
// may have further to go.  Written out as one block with its own branches: a
// compare finds most pairs in order in all 64 lanes, a slot that moved is the
// only one that can move on, and the compiler sees straight-line code (the
// same chain as nested ifs spilled 190 registers at 20 slots).
template <int N, int K>
__device__ __forceinline__ void slots_sink(Slots<N>& sl, uint64_t& deep) {
    uint64_t all;
    if constexpr (K == 1) {
        asm volatile(
            "v_cmp_gt_f32 vcc, %[a0], %[b0]\n\t"
            "s_cbranch_vccz .Lord%=\n\t"
            "s_and_saveexec_b64 %[all], vcc\n\t"
            "v_swap_b32 %[a0], %[b0]\n\t"
            "v_swap_b32 %[a1], %[b1]\n\t"
            "v_swap_b32 %[a2], %[b2]\n\t"
            "s_mov_b64 exec, %[all]\n"
            ".Lord%=:"
            : [a0] "+v"(sl.d[0]), [a1] "+v"(sl.rec[0]), [a2] "+v"(sl.s[0]), [b0] "+v"(sl.d[1]),
              [b1] "+v"(sl.rec[1]), [b2] "+v"(sl.s[1]), [all] "=&s"(all)
            :
            : "vcc", "scc");
    } else if constexpr (K == 2) {
        asm volatile(
            "v_cmp_gt_f32 vcc, %[b0], %[c0]\n\t"
            "s_cbranch_vccz .Lord%=\n\t"
            "s_and_saveexec_b64 %[all], vcc\n\t"
            "v_swap_b32 %[b0], %[c0]\n\t"
            "v_swap_b32 %[b1], %[c1]\n\t"
            "v_swap_b32 %[b2], %[c2]\n\t"
            "v_cmp_gt_f32 vcc, %[a0], %[b0]\n\t"
            "s_cbranch_vccz .Lend%=\n\t"
            "s_mov_b64 exec, vcc\n\t"
            "v_swap_b32 %[a0], %[b0]\n\t"
            "v_swap_b32 %[a1], %[b1]\n\t"
            "v_swap_b32 %[a2], %[b2]\n"
            ".Lend%=:\n\t"
            "s_mov_b64 exec, %[all]\n"
            ".Lord%=:"
            : [a0] "+v"(sl.d[0]), [a1] "+v"(sl.rec[0]), [a2] "+v"(sl.s[0]), [b0] "+v"(sl.d[1]),
              [b1] "+v"(sl.rec[1]), [b2] "+v"(sl.s[1]), [c0] "+v"(sl.d[2]),
              [c1] "+v"(sl.rec[2]), [c2] "+v"(sl.s[2]), [all] "=&s"(all)
            :
            : "vcc", "scc");
    } else {
        asm volatile(
            "v_cmp_gt_f32 vcc, %[c0], %[d0]\n\t"
            "s_cbranch_vccz .Lord%=\n\t"
            "s_and_saveexec_b64 %[all], vcc\n\t"
            "v_swap_b32 %[c0], %[d0]\n\t"
            "v_swap_b32 %[c1], %[d1]\n\t"
            "v_swap_b32 %[c2], %[d2]\n\t"
            "v_cmp_gt_f32 vcc, %[b0], %[c0]\n\t"
            "s_cbranch_vccz .Lend%=\n\t"
            "s_mov_b64 exec, vcc\n\t"
            "v_swap_b32 %[b0], %[c0]\n\t"
            "v_swap_b32 %[b1], %[c1]\n\t"
            "v_swap_b32 %[b2], %[c2]\n\t"
            "v_cmp_gt_f32 vcc, %[a0], %[b0]\n\t"
            "s_cbranch_vccz .Lend%=\n\t"
            "s_mov_b64 exec, vcc\n\t"
            "v_swap_b32 %[a0], %[b0]\n\t"
            "v_swap_b32 %[a1], %[b1]\n\t"
            "v_swap_b32 %[a2], %[b2]\n\t"
            "s_or_b64 %[deep], %[deep], vcc\n"
            ".Lend%=:\n\t"
            "s_mov_b64 exec, %[all]\n"
            ".Lord%=:"
            : [a0] "+v"(sl.d[K - 3]), [a1] "+v"(sl.rec[K - 3]), [a2] "+v"(sl.s[K - 3]),
              [b0] "+v"(sl.d[K - 2]), [b1] "+v"(sl.rec[K - 2]), [b2] "+v"(sl.s[K - 2]),
              [c0] "+v"(sl.d[K - 1]), [c1] "+v"(sl.rec[K - 1]), [c2] "+v"(sl.s[K - 1]),
              [d0] "+v"(sl.d[K]), [d1] "+v"(sl.rec[K]), [d2] "+v"(sl.s[K]), [all] "=&s"(all),
              [deep] "+s"(deep)
            :
            : "vcc", "scc");
    }
}

template <int N, int K, int A>
__device__ __forceinline__ void slots_sink_all(Slots<N>& sl, uint64_t& deep) {
    if constexpr (K < A) {
        slots_sink<N, K>(sl, deep);
        slots_sink_all<N, K + 1, A>(sl, deep);
    }
}

// Puts the A lowest slots of every lane in order of position (equal positions
// in either order).  A pass in which no slot moved three places leaves them
// in order: each slot it moved sank into an ordered run below it.
template <int N, int A>
__device__ __forceinline__ void slots_sort(Slots<N>& sl) {
    uint64_t deep;
    do {
        deep = 0;
        slots_sink_all<N, 1, A>(sl, deep);
    } while (__builtin_amdgcn_readfirstlane((uint32_t)deep | (uint32_t)(deep >> 32)));
}

// Steps 1-4 of a plain tick for the A lowest slots (the others are parked in
// every lane), without the test for the line.  Bottom up, so that a slot's
// step overwrites the one before only after the slot below has read it.
// kKeep leaves each competitor's start-of-tick position in the place of its
// draw, for the crossing fractions.
template <int N, Pace kPace, int A, bool kKeep>
__device__ __forceinline__ void slots_tick_plain(Slots<N>& sl, const float (&gap)[N],
                                                 uint32_t ucol, uint32_t pbase, uint32_t t,
                                                 uint32_t sim, uint32_t request, uint32_t k0,
                                                 uint32_t k1) {
    if constexpr (kPace == kPaceTable) write_pace_terms<N>(pbase, t);
    write_draws<N>(ucol, t, sim, request, k0, k1);
    const uint32_t ubias = ucol - 16u * pbase;
    constexpr int kPf = 4;
    float pu[N], pth[N], pga[N];
    f32x4 pp[N];
    auto fetch = [&](int k) {
        const uint32_t rec = sl.rec[k];
        pu[k] = lds_ld<float>(ubias + (rec << 4));
        if constexpr (kKeep) lds_st<float>(ubias + (rec << 4), sl.d[k]);
        pp[k] = lds_ld<f32x4>(rec);
        if constexpr (kPace == kPaceTable) {
            const f32x2 q = lds_ld<f32x2>(rec + kRecHalf<N>);
            pth[k] = q.x;
            pga[k] = q.y;
        } else {
            pth[k] = lds_ld<float>(rec + kRecHalf<N>);
        }
    };
#pragma unroll
    for (int k = 0; k < A && k < kPf; ++k) fetch(k);
#pragma unroll
    for (int k = 0; k < A; ++k) {
        if (k + kPf < A) fetch(k + kPf);
        const float d = sl.d[k];
        const f32x4 p = pp[k];
        float R = p.z + p.w * d;
        if constexpr (kPace == kPaceTable) R = R + pga[k];
        float f = p.x + p.y * pu[k];
        if (k < A - 1) {
            const float s_min = __uint_as_float(
                min(__float_as_uint(sl.s[k]), __float_as_uint(sl.s[k + 1])));
            f = (gap[k] <= pth[k]) ? s_min : f;
        }
        const float S = R * f;
        sl.d[k] = d + S;
        sl.s[k] = S;
    }
}

// Slot K's test for the line, in every lane: where its position has reached
// it, the slot is parked and its bit set in `cross`; `kset` collects the slots
// of which some lane crossed.
template <int N, int K>
__device__ __forceinline__ void slots_cross(Slots<N>& sl, float L, uint32_t& cross,
                                            uint32_t& kset) {
    uint64_t all;
    asm volatile(
        "v_cmp_le_f32 vcc, %[line], %[d]\n\t"
        "s_cbranch_vccz .Lnone%=\n\t"
        "s_and_saveexec_b64 %[all], vcc\n\t"
        "v_or_b32 %[cross], %[bit], %[cross]\n\t"
        "v_mov_b32 %[d], 0x7fc00000\n\t"
        "s_or_b32 %[kset], %[kset], %[bit]\n\t"
        "s_mov_b64 exec, %[all]\n"
        ".Lnone%=:"
        : [d] "+v"(sl.d[K]), [cross] "+v"(cross), [kset] "+s"(kset), [all] "=&s"(all)
        : [line] "s"(L), [bit] "i"(1u << K)
        : "vcc", "scc");
}

template <int N, int K, int A>
__device__ __forceinline__ void slots_cross_all(Slots<N>& sl, float L, uint32_t& cross,
                                                uint32_t& kset) {
    if constexpr (K < A) {
        slots_cross<N, K>(sl, L, cross, kset);
        slots_cross_all<N, K + 1, A>(sl, L, cross, kset);
    }
}

// Step 5 after a plain tick: ranks a lane's finishers of this tick (`cross`:
// their slots, parked by slots_cross; `kset`: those of the whole wave) as
// slots_rank_park does.  The crossing fraction of competitor c goes to its own
// place of the draw table, where slots_tick_plain left its start-of-tick
// position.
template <int N, int A, class Win>
__device__ __forceinline__ int slots_rank(const Slots<N>& sl, uint32_t cross, uint32_t kset,
                                          bool rank, float L, uint32_t ucol, uint32_t icol,
                                          uint32_t pbase, int nfin, const Win& win, uint32_t row) {
    const int c = __builtin_popcount(cross);
#pragma unroll
    for (int k = 0; k < A; ++k)
        if ((kset >> k) & 1u) {  // the same in every lane
            if (rank && ((cross >> k) & 1u)) {
                const uint32_t j = __builtin_popcount(cross & ((1u << k) - 1u));
                const uint32_t off = sl.rec[k] - pbase;
                lds_st<uint8_t>(icol + 64u * j, (uint8_t)(off >> 4));
                // a lone finisher needs no fraction
                if (c > 1) {
                    const uint32_t place = ucol + 16u * off;
                    lds_st<float>(place, (L - lds_ld<float>(place)) / sl.s[k]);
                }
            }
        }
    if (!rank) return 0;
    uint32_t used = 0u;
    for (int r = 0; r < c; ++r) {
        int bj = -1;
        float bf = 0.0f;
        uint32_t bid = 0u;
        for (int j = 0; j < c; ++j) {
            const uint32_t id = lds_ld<uint8_t>(icol + 64u * j);
            const float f = lds_ld<float>(ucol + 256u * id);
            const bool better =
                !((used >> j) & 1u) && ((bj < 0) || (f < bf) || (f == bf && id < bid));
            bj = better ? j : bj;
            bf = better ? f : bf;
            bid = better ? id : bid;
        }
        used |= 1u << bj;  // c - r > 0 entries are unused, so bj >= 0
        const int rr = nfin + r;
        if (rr == 0) win(bid);
        if (row != kNoRow) lds_st<uint8_t>(row + rr, (uint8_t)bid);
    }
    return c;
}

// How a run of ticks ended.
enum Outcome : int { kEnded = 0, kParked = 1, kTied = 2 };

// Runs f(std::integral_constant<int, A>) for A = N, N - kStep, ... (A >=
// kStep > 0; A = N only where kStep = 0) one after the other for as long as f
// returns kParked.
template <int A, int kStep, class F>
__device__ __forceinline__ Outcome run_phases(F& f) {
    const Outcome o = f(std::integral_constant<int, A>{});
    if constexpr (kStep > 0 && A - kStep >= kStep)
        if (o == kParked) return run_phases<A - kStep, kStep>(f);
    return o;
}

// One generation: up to 64 simulations of one race from one state, one per
// lane, in lockstep from tick t0.  `live` marks the lanes that hold a
// simulation; sim_of(lane) and request_of(lane) are its index and its request
// id; `rows` (or kNoRow) is the LDS table of their finish orders, N bytes a
// lane; `ubase` and `ibase` locate the wave's draw and finisher-id tables.
// Lanes whose simulation has ended keep stepping with the others (their
// results are no longer recorded), so the tick needs no divergent branch.
// win(c) is told each simulation's winner; competitor-steps add to `steps`.
// kSkipStep > 0 stops stepping and sorting the top slots once they are
// parked in every lane, kSkipStep slots at a time (a copy of the tick per
// active count): late in a generation most lanes have parked most of their
// competitors.
template <int N, Pace kPace, int kSkipStep, class Sim, class Request, class Win>
__device__ __forceinline__ void run_generation(uint32_t ubase, uint32_t ibase, uint32_t pbase,
                                               float L, const StepBounds& sb,
                                               const float* __restrict__ d0,
                                               const float* __restrict__ s0,
                                               const uint8_t* __restrict__ id0, uint32_t t0,
                                               bool live, const Sim& sim_of,
                                               const Request& request_of,
                                               uint32_t k0, uint32_t k1, int stop_after,
                                               uint32_t rows, const Win& win,
                                               unsigned long long& steps) {
    Slots<N> sl;
    slots_reset<N>(sl, d0, s0, id0, pbase);
    uint32_t t = t0;
    int nfin = 0;
    uint32_t run = 0;  // this lane's competitor-steps (at most N * 2^20)
    auto row_of = [&](uint32_t lane) {
        return rows == kNoRow ? kNoRow : rows + (uint32_t)N * lane;
    };
    // Counts this tick's `k` finishers and settles the simulations that end.
    auto end_tick = [&](int k) {
        nfin += k;
        run += (uint32_t)k * (t + 1 - t0);
        if (live && (nfin >= stop_after || t + 1 - t0 >= kTickLimit)) {
            if (rows != kNoRow) {
                const uint32_t row = row_of(lane_here());
                for (int r = nfin; r < N; ++r) lds_st<uint8_t>(row + r, 0xFF);
            }
            run += (uint32_t)(N - nfin) * (t + 1 - t0);
            live = false;
        }
    };
    // Plain ticks in which nobody can reach the line, for as long as there
    // are any; afterwards `may_open` tells whether there can be more.
    bool may_open = true;
    auto open_run = [&]() {
        // what depends on the simulation index only is computed once per run
        // of open ticks, and not kept across the other ticks
        const uint32_t lane = lane_here();
        const uint32_t sim = sim_of(lane), request = request_of(lane);
        float gap[N];
        bool tie = slots_gaps<N, N>(sl, gap);
        int left = t - t0 < kTickLimit - 16u ? open_ticks<N>(sl, L, sb) : 0;
        while (left != 0 && !tie) {
            t = __builtin_amdgcn_readfirstlane(t);  // the wave's: the compiler cannot tell
            slots_tick_plain<N, kPace, N, false>(sl, gap, ubase + 4u * lane_here(), pbase, t, sim,
                                                 request, k0, k1);
            t += 1;
            slots_sort<N, N>(sl);
            tie = slots_gaps<N, N>(sl, gap);
            left = __builtin_amdgcn_readfirstlane(left) - 1;
            if (left == 0 && t - t0 < kTickLimit - 16u) left = open_ticks<N>(sl, L, sb);
        }
        may_open = left != 0;
    };
    // One phase runs plain ticks of the A lowest slots (slots A .. N-1 are
    // parked in every lane) until the generation ends, a tie, or until the
    // next kSkipStep slots down are parked in every lane too.
    auto phase = [&](auto act) -> Outcome {
        constexpr int A = decltype(act)::value;
        // the slots are in order, so a lane's parked ones are its top ones:
        // the next kSkipStep down are parked everywhere iff the lowest is
        auto parked_below = [&]() {
            if constexpr (kSkipStep > 0 && A - kSkipStep >= kSkipStep)
                return !__builtin_amdgcn_ballot_w64(__float_as_uint(sl.d[A - kSkipStep]) !=
                                                    __float_as_uint(parked()));
            return false;
        };
        if (parked_below()) return kParked;
        float gap[N];
        bool tie = slots_gaps<N, A>(sl, gap);
        while (!tie) {
            if (!__builtin_amdgcn_ballot_w64(live)) return kEnded;
            t = __builtin_amdgcn_readfirstlane(t);  // the wave's: the compiler cannot tell
            const uint32_t lane = lane_here(), ucol = ubase + 4u * lane;
            slots_tick_plain<N, kPace, A, true>(sl, gap, ucol, pbase, t, sim_of(lane),
                                                request_of(lane), k0, k1);
            slots_sort<N, A>(sl);
            uint32_t cross = 0u, kset = 0u;
            slots_cross_all<N, 0, A>(sl, L, cross, kset);
            kset = __builtin_amdgcn_readfirstlane(kset);
            int k = 0;
            if (kset)
                k = slots_rank<N, A>(sl, cross, kset, live && cross, L, ucol,
                                     ibase + lane, pbase, nfin, win, row_of(lane));
            end_tick(k);
            t += 1;
            if (kset && parked_below()) return kParked;
            tie = slots_gaps<N, A>(sl, gap);
        }
        return kTied;
    };
    for (;;) {
        if (may_open) open_run();
        if (run_phases<N, kSkipStep>(phase) == kEnded) break;
        // a tie: ticks that look past equal positions, in index order, until
        // the positions differ again
        slots_opaque<N>(sl);
        slots_restore<N>(sl);
        do {
            t = __builtin_amdgcn_readfirstlane(t);
            const uint32_t lane = lane_here(), ucol = ubase + 4u * lane;
            const uint32_t cross =
                slots_tick<N, kPace>(sl, ucol, pbase, L, t, sim_of(lane), request_of(lane), k0,
                                     k1);
            int k = 0;
            if (__builtin_amdgcn_ballot_w64(cross != 0u))
                k = slots_rank_park<N>(sl, cross, live && cross, L, ucol, ibase + lane, pbase,
                                       nfin, win, row_of(lane));
            end_tick(k);
            t += 1;
            slots_restore<N>(sl);
            slots_opaque<N>(sl);  // (after the loop, the other loops spilled)
        } while (__builtin_amdgcn_ballot_w64(live) && slots_tied<N>(sl));
    }
    steps += run;
}

}  // namespace bbe
