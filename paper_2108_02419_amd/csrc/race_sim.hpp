// race_sim.hpp -- one simulated race per lane, 64 lanes in lockstep
// (paper Section 3, Eq. 1).
//
// Layout.  A lane keeps its competitors in N register "slots" sorted by
// position (ascending; finished competitors are parked at the top with a
// NaN position).  Slot k holds the position d[k], the LDS byte offset
// rec[k] of its competitor's parameter record (pbase + 16 * competitor
// index; it also locates the competitor's draw) and the previous step s[k].
// The competitor ahead of slot k is then the first slot above it with a larger
// position -- slot k+1 unless positions are equal -- and the query of Eq. 1
// costs O(1) per competitor instead of a scan over all pairs.
//
// One tick (all 64 lanes at the same absolute tick t):
//   1. draws in competitor order: Philox4x32-10(key = seed,
//      ctr = (t, sim, request, b)) for blocks b = 0 .. ceil(N/8)-1;
//      competitor c takes word (c>>1)&3 of block c>>3, its high half for
//      even c and its low half for odd c, as the integer k (u = k * 2^-16);
//      the draws go to the lane's column of an LDS table and each slot
//      reads the draw of its own competitor (write_draws, SlotInputs);
//   2. competitor ahead: the running competitor with the smallest position
//      greater than d_c (lowest index among equal positions); gap =
//      fl(d_ahead - d_c), +inf if nobody is ahead;
//   3. Eq. 1: R = alpha + beta*d (+ gamma*min(t, tau) in the paced
//      variants); free: S = R*(elo + espan*u); blocked (gap <= theta):
//      S = R*min(s_c, s_ahead);
//   4. synchronous update d += S, s = S of the running competitors
//      (slots_tick_plain, slots_tick_tied), and the slots' order restored
//      (slots_sort);
//   5. a competitor whose position has reached L has crossed the line and is
//      parked (slots_cross; position NaN: every comparison with it is false, so
//      a parked slot never crosses again and is never "ahead" of anyone); this
//      tick's finishers are ranked after the earlier ones, among themselves by
//      the fraction fl((L - d_old)/S), then by index (slots_rank).
//
// Ticks come in three kinds, each a loop of its own (run_generation): open ones,
// in which nobody can reach the line (no step 5), plain ones, and those in which
// some lane has equal positions.
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

// ---------------------------------------------------------------------------
// Plain ticks: no two running competitors of a lane share a position.  Nearly
// every tick of a wave is plain (equal positions: the start line, and a few
// ticks in ten thousand after it): the competitor ahead of slot k is slot k+1
// itself, and float compares order the slots (no compare with a parked slot's NaN
// holds, which leaves the parked slots at the top and whoever leads unblocked).
//
// With one kind of tick for all, which looked past equal positions and ordered
// the slots by (position, index) in 64-bit compares, the straight-line block at 20
// competitors had 466 vector instructions against 313 of an open tick.  The
// kernels are bound by vector issue (98% busy over the uneven batch), so that is
// the gain: 10^6 simulations of 20 competitors from the start 7.54 -> 5.93 ms, 4096
// uneven in-play requests 19.95 -> 16.4 ms.  Fields that stay tied for good take
// the loop of slots_tick_tied throughout: 4*10^5 simulations of 20 identical
// competitors 2.24 -> 2.11 ms against that one kind, 10^5 of two 154 -> 161 us.
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

// What a tick reads of the slots' competitors, from the LDS tables: the draw of
// competitor c sits at ucol + 256*c = ubias + 16*rec.
template <int N, Pace kPace>
struct SlotInputs {
    float draw[N], theta[N], term[N];
    f32x4 par[N];  // elo, espan16, alpha, beta
    // kKeep: the slot's position takes the place of the draw
    template <bool kKeep>
    __device__ __forceinline__ void fetch(const Slots<N>& sl, int k, uint32_t ubias) {
        const uint32_t rec = sl.rec[k];
        draw[k] = lds_ld<float>(ubias + (rec << 4));
        if constexpr (kKeep) lds_st<float>(ubias + (rec << 4), sl.d[k]);
        par[k] = lds_ld<f32x4>(rec);
        if constexpr (kPace == kPaceTable) {
            const f32x2 q = lds_ld<f32x2>(rec + kRecHalf<N>);
            theta[k] = q.x;
            term[k] = q.y;
        } else {
            theta[k] = lds_ld<float>(rec + kRecHalf<N>);
        }
    }
    __device__ __forceinline__ float response(int k, float d) const {  // R of Eq. 1
        const float R = par[k].z + par[k].w * d;
        if constexpr (kPace == kPaceTable) return R + term[k];
        return R;
    }
    __device__ __forceinline__ float free(int k) const {  // a free step over R
        return par[k].x + par[k].y * draw[k];
    }
};

// Steps 1-4 of a plain tick for the A lowest slots (the others are parked in
// every lane), without the test for the line.  Bottom up, so that a slot's
// step overwrites the one before only after the slot below has read it.
// kKeep leaves each competitor's start-of-tick position in the place of its
// draw, for the crossing fractions.
template <int N, Pace kPace, int A, bool kKeep>
__device__ __forceinline__ void slots_tick_plain(Slots<N>& sl, const float (&gap)[N],
                                                 uint32_t ucol, uint32_t pbase) {
    const uint32_t ubias = ucol - 16u * pbase;
    constexpr int kPf = 4;
    SlotInputs<N, kPace> in;
#pragma unroll
    for (int k = 0; k < A && k < kPf; ++k) in.template fetch<kKeep>(sl, k, ubias);
#pragma unroll
    for (int k = 0; k < A; ++k) {
        if (k + kPf < A) in.template fetch<kKeep>(sl, k + kPf, ubias);
        // keeps the reads that far ahead: left to itself the compiler had 28 waits
        // for all of LDS in the open tick of 17 competitors (5 to 14 from 13 to
        // 16), 8% of a tick where a SIMD has one wave
        if constexpr (!kKeep) __builtin_amdgcn_sched_barrier(0);
        const float d = sl.d[k];
        float f = in.free(k);
        if (k < A - 1) {
            const float s_min = __uint_as_float(
                min(__float_as_uint(sl.s[k]), __float_as_uint(sl.s[k + 1])));
            f = (gap[k] <= in.theta[k]) ? s_min : f;
        }
        const float S = in.response(k, d) * f;
        sl.d[k] = d + S;
        sl.s[k] = S;
    }
}

// Puts the equal positions of slots K and K + 1 in index order in every lane;
// `equal` collects the lanes that have some, `moved` those that were not in order.
template <int N, int K>
__device__ __forceinline__ void slots_order_pair(Slots<N>& sl, uint64_t& equal, uint64_t& moved) {
    uint64_t all;
    asm volatile(
        "v_cmp_eq_f32 vcc, %[a0], %[b0]\n\t"
        "s_cbranch_vccz .Ldiff%=\n\t"
        "v_cmp_gt_u32 %[all], %[a1], %[b1]\n\t"
        "s_or_b64 %[equal], %[equal], vcc\n\t"
        "s_and_b64 vcc, vcc, %[all]\n\t"
        "s_cbranch_scc0 .Ldiff%=\n\t"
        "s_mov_b64 %[all], exec\n\t"
        "s_mov_b64 exec, vcc\n\t"
        "v_swap_b32 %[a1], %[b1]\n\t"
        "v_swap_b32 %[a2], %[b2]\n\t"
        "s_or_b64 %[moved], %[moved], vcc\n\t"
        "s_mov_b64 exec, %[all]\n"
        ".Ldiff%=:"
        : [a1] "+v"(sl.rec[K]), [a2] "+v"(sl.s[K]), [b1] "+v"(sl.rec[K + 1]),
          [b2] "+v"(sl.s[K + 1]), [all] "=&s"(all), [equal] "+s"(equal), [moved] "+s"(moved)
        : [a0] "v"(sl.d[K]), [b0] "v"(sl.d[K + 1])
        : "vcc", "scc");
}

template <int N, int K, int A>
__device__ __forceinline__ void slots_order_pairs(Slots<N>& sl, uint64_t& equal, uint64_t& moved) {
    if constexpr (K + 1 < A) {
        slots_order_pair<N, K>(sl, equal, moved);
        slots_order_pairs<N, K + 1, A>(sl, equal, moved);
    }
}

// Puts equal positions among the A lowest slots in index order (positions being
// in order), in every lane; whether there are any.
template <int N, int A>
__device__ __forceinline__ bool slots_order_equal(Slots<N>& sl) {
    uint64_t equal, moved;
    do {
        equal = moved = 0;
        slots_order_pairs<N, 0, A>(sl, equal, moved);
    } while (A > 2 && __builtin_amdgcn_readfirstlane((uint32_t)moved | (uint32_t)(moved >> 32)));
    return __builtin_amdgcn_readfirstlane((uint32_t)equal | (uint32_t)(equal >> 32));
}

// slots_tick_plain, with kKeep, where some lane has equal positions (in index
// order).  The competitor ahead of slot k is then the first slot above it with a
// larger position: slot k+1, or -- where positions are equal -- the one found for
// slot k+1, carried down in (nd, ns).  Top down, the start-of-tick position and
// step of slot k+1 in (d_up, s_up).
template <int N, Pace kPace, int A>
__device__ __forceinline__ void slots_tick_tied(Slots<N>& sl, uint32_t ucol, uint32_t pbase) {
    const uint32_t ubias = ucol - 16u * pbase;
    constexpr int kPf = 4;
    SlotInputs<N, kPace> in;
#pragma unroll
    for (int k = A - 1; k >= 0 && k >= A - kPf; --k) in.template fetch<true>(sl, k, ubias);
    float nd = __builtin_inff(), ns = 0.0f;
    float d_up = __builtin_inff(), s_up = 0.0f;
#pragma unroll
    for (int k = A - 1; k >= 0; --k) {
        if (k - kPf >= 0) in.template fetch<true>(sl, k - kPf, ubias);
        const float d = sl.d[k], s = sl.s[k];
        const bool gt = d_up > d;  // false next to a parked (NaN) slot
        nd = gt ? d_up : nd;
        ns = gt ? s_up : ns;
        const float s_min =
            __uint_as_float(min(__float_as_uint(s), __float_as_uint(ns)));
        const float S = in.response(k, d) * ((nd - d <= in.theta[k]) ? s_min : in.free(k));
        sl.d[k] = d + S;
        sl.s[k] = S;
        d_up = d;
        s_up = s;
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

template <int N, int K, int M>
__device__ __forceinline__ void slots_cross_few(Slots<N>& sl, float L, uint32_t& cross,
                                                uint32_t& kset) {
    if constexpr (M > 0 && K >= 0) {
        slots_cross<N, K>(sl, L, cross, kset);
        slots_cross_few<N, K - 1, M - 1>(sl, L, cross, kset);
    }
}

// Slots from the top down, a few at a time (positions being in order): below one
// that is short of the line in every lane nobody is at it.
constexpr int kCrossStep = 5;
template <int N, int K>
__device__ __forceinline__ void slots_cross_all(Slots<N>& sl, float L, uint32_t& cross,
                                                uint32_t& kset) {
    if constexpr (K >= 4)
        if (!__builtin_amdgcn_ballot_w64(!(sl.d[K] < L))) return;
    slots_cross_few<N, K, kCrossStep>(sl, L, cross, kset);
    if constexpr (K >= kCrossStep) slots_cross_all<N, K - kCrossStep>(sl, L, cross, kset);
}

// Ranks a lane's finishers of this tick (`cross`: their slots, parked by
// slots_cross; `kset`: those of the whole wave) after the `nfin` earlier ones and
// records them; returns the number ranked.  `rank` is false in lanes whose
// simulation has already ended, and in those without a finisher.  Entry j (the
// j-th set bit of `cross`) holds its competitor index in the lane's column of a
// byte table, at icol + 64*j; the crossing fraction of competitor c goes to its
// own place of the draw table, where the tick left its start-of-tick position.
// The entries are then picked in (fraction, index) order, so the work grows with
// c^2 for the few finishers of a tick rather than with c*N.
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
enum Outcome : int { kEnded = 0, kParked = 1, kTurn = 2 };

// The active slots of the phase after one of A: kStep less (0: there is none),
// for ticks of equal positions twice that in large fields, which keeps the
// copies of their rarer loop few.
template <int kStep, bool kTied>
constexpr int next_phase(int A) {
    const int less = kTied && A > 4 * kStep ? 2 * kStep : kStep;
    return kStep > 0 && A - less >= kStep ? A - less : 0;
}

// Runs f(A, kTied) as constants for A = N and each next phase one after the other
// for as long as f returns kParked.
template <int A, int kStep, bool kTied, class F>
__device__ __forceinline__ Outcome run_phases(F& f) {
    const Outcome o =
        f(std::integral_constant<int, A>{}, std::integral_constant<bool, kTied>{});
    if constexpr (next_phase<kStep, kTied>(A) > 0)
        if (o == kParked) return run_phases<next_phase<kStep, kTied>(A), kStep, kTied>(f);
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
    // Counts this tick's `k` finishers and settles the simulations that end
    // (nobody's does in a tick without finishers, but at the tick limit).
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
            const uint32_t ucol = ubase + 4u * lane_here();
            if constexpr (kPace == kPaceTable) write_pace_terms<N>(pbase, t);
            write_draws<N>(ucol, t, sim, request, k0, k1);
            slots_tick_plain<N, kPace, N, false>(sl, gap, ucol, pbase);
            t += 1;
            slots_sort<N, N>(sl);
            tie = slots_gaps<N, N>(sl, gap);
            left = __builtin_amdgcn_readfirstlane(left) - 1;
            if (left == 0 && t - t0 < kTickLimit - 16u) left = open_ticks<N>(sl, L, sb);
        }
        may_open = left != 0;
    };
    // One phase runs ticks of the A lowest slots (slots A .. N-1 are parked in
    // every lane), plain ones until positions are equal or, kTied, those of equal
    // positions until there are none; or until the generation ends, or more slots
    // are parked in every lane.
    auto phase = [&](auto act, auto tied) -> Outcome {
        constexpr int A = decltype(act)::value;
        constexpr bool kTied = decltype(tied)::value;
        constexpr int kNext = next_phase<kSkipStep, kTied>(A);
        // the slots are in order, so a lane's parked ones are its top ones:
        // all down to slot kNext are parked everywhere iff that one is
        auto parked_below = [&]() {
            if constexpr (kNext > 0)
                return !__builtin_amdgcn_ballot_w64(__float_as_uint(sl.d[kNext]) !=
                                                    __float_as_uint(parked()));
            return false;
        };
        if (parked_below()) return kParked;
        float gap[N];
        auto looks = [&]() {  // whether the next tick is of the other kind
            if constexpr (kTied) return !slots_order_equal<N, A>(sl);
            return slots_gaps<N, A>(sl, gap);
        };
        // what depends on the simulation index only is computed once where there
        // are registers for it
        constexpr bool kOnce = kSkipStep == 0;
        uint32_t sim0 = 0, request0 = 0;
        if constexpr (kOnce) {
            sim0 = sim_of(lane_here());
            request0 = request_of(lane_here());
        }
        // (at least one tick where the other kind sent it here)
        bool turn = looks() && !kTied;
        if (!__builtin_amdgcn_ballot_w64(live)) return kEnded;
        while (!turn) {
            t = __builtin_amdgcn_readfirstlane(t);  // the wave's: the compiler cannot tell
            const uint32_t lane = lane_here(), ucol = ubase + 4u * lane;
            if constexpr (kPace == kPaceTable) write_pace_terms<N>(pbase, t);
            write_draws<N>(ucol, t, kOnce ? sim0 : sim_of(lane),
                           kOnce ? request0 : request_of(lane), k0, k1);
            if constexpr (kTied)
                slots_tick_tied<N, kPace, A>(sl, ucol, pbase);
            else
                slots_tick_plain<N, kPace, A, true>(sl, gap, ucol, pbase);
            slots_sort<N, A>(sl);
            uint32_t cross = 0u, kset = 0u;
            slots_cross_all<N, A - 1>(sl, L, cross, kset);
            kset = __builtin_amdgcn_readfirstlane(kset);
            if (kset || t + 1 - t0 >= kTickLimit) {
                end_tick(slots_rank<N, A>(sl, cross, kset, live && cross, L, ucol, ibase + lane,
                                          pbase, nfin, win, row_of(lane)));
                if (!__builtin_amdgcn_ballot_w64(live)) return kEnded;
            }
            t += 1;
            if (kset && parked_below()) return kParked;
            turn = looks();
        }
        return kTurn;
    };
    for (;;) {
        if (may_open) open_run();
        if (run_phases<N, kSkipStep, false>(phase) == kEnded) break;
        if (run_phases<N, kSkipStep, true>(phase) == kEnded) break;
    }
    steps += run;
}

}  // namespace bbe
