// FP64 near field of one wavefront: a few sinks of one leaf against a slice of
// the leaf's sources (device code only; used by the force and by the jerk
// direct sums).
//
// The sinks sit in scalar registers and the 64 lanes hold 64 consecutive
// sources of the leaf's concatenated range list, so every lane works on every
// pair, one source load serves all the sinks, and a source coordinate minus a
// sink coordinate is one instruction with a scalar operand.  Each sink's sum
// stays spread over the lanes until the end of the slice, where the lanes are
// added once.  What bounds it is VALU issue: 16 FP64 operations and a
// quarter-rate reciprocal square root per pair, 20 issue slots; 22.4 are
// issued, 95% of the kernel's cycles.  Measured at N = 10^6 Plummer (1.47e10
// pairs, leaves of 23 particles on average): 10.2 ms, 1.44e12 pairs/s, against
// 12.9 ms for two sinks per lane with strided phases (26 slots per pair: lanes
// idle in uneven groups, a load per two pairs); the short lists of the sink-scale
// estimate at N = 10^5: 75 us against 214 us.  Loading the next step's source
// ahead costs registers and moves and is slower (by 0.7 ms): four wavefronts per
// SIMD cover the load.  The lists are flattened once per leaf by the plan:
// flattening them in each wavefront took 1.2 ms more.
//
// The order in which a sink's sources are added depends only on its leaf's
// lists (lane = position in the list modulo 64, slices of NEAR_TASK sources,
// lanes added in a fixed pattern), not on how many sinks share the wavefront,
// so calls that share a leaf's lists agree bit for bit.
#pragma once

#include <climits>

#include "internal.h"
#include "lanes.h"

namespace fmm {

// the value lane l holds, in scalar registers
__device__ __forceinline__ double readlane_f64(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Sinks are dealt evenly to the groups of a leaf: group g of ngroups holds
// the sinks [group_begin(g), group_begin(g + 1)) of nb; group_of is its inverse.
__device__ __forceinline__ int group_begin(int nb, int ngroups, int g) {
    return (int)((int64_t)g * nb / ngroups);
}
__device__ __forceinline__ int group_of(int nb, int ngroups, int k) {
    return (int)((((int64_t)k + 1) * ngroups - 1) / nb);
}

// One wavefront's task: sinks [sb, sb + r) of a leaf, `count` sources of the
// leaf's list from position j0 on; first: the list entry that holds j0 (an
// index into the entries of its part); single: the leaf's only slice.
struct NearTask {
    int sb, first, j0, r, count;
    bool single;
};
__device__ __forceinline__ int4 pack_task(int sb, int first, int j0, int r, int count,
                                          bool single) {
    static_assert(NEAR_R < 16 && NEAR_JERK_R < 16 && NEAR_TASK < (1 << 26), "fields of w");
    return make_int4(sb, first, j0, r | (single ? 16 : 0) | (count << 5));
}
__device__ __forceinline__ NearTask unpack_task(int4 v) {
    const int w = __builtin_amdgcn_readfirstlane(v.w);
    return {__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
            __builtin_amdgcn_readfirstlane(v.z), w & 15, w >> 5, (w & 16) != 0};
}

// Runs over the sources of a task, 64 per step.  load(i) fetches source
// particle i; fast(src) adds 64 sources none of which
// is one of the sinks; checked(src, i, on) adds those of the lanes with on set,
// i being their particle index (steps that touch the sinks themselves, and the
// last step of a list).  entry: the leaf's ranges as (shift, end), position j
// of the list before `end` being particle j + shift, closed by an entry with
// end = INT_MAX whose shift makes the at most 127 positions past the list
// particles 0..127 (the arrays that load reads are padded for that).  Each lane
// follows its own entry q of the 64 held by the wavefront.
template <class Load, class Fast, class Checked>
__device__ __forceinline__ void near_sources(const int2 *entry, const NearTask &t, Load &&load,
                                             Fast &&fast, Checked &&checked) {
    const int lane = lane_id();
    int base = t.first;
    int shift0, end0;
    auto fetch = [&]() {          // 64 entries from base on
        const int2 v = entry[base + lane];
        shift0 = v.x;
        const unsigned long long last = __ballot(v.y == INT_MAX);
        // what follows the closing entry belongs to another leaf
        end0 = last && lane > __ffsll((long long)last) - 1 ? INT_MAX : v.y;
    };
    fetch();
    // q: byte index 4 * (entry) of the lane's entry, as the lane exchange takes it
    auto pick = [&](int at, int v) { return __builtin_amdgcn_ds_bpermute(at, v); };
    // the entry of this lane's first position: those that end before it precede
    int j = t.j0 + lane, q = 0;
#pragma unroll
    for (int s = FMM_WAVE / 2; s > 0; s >>= 1)
        if (pick(q + 4 * (s - 1), end0) <= j) q += 4 * s;
    int e = pick(q, end0), sh = pick(q, shift0);
    // on to the next 64 positions.  A range holds at least one particle, so the
    // lanes' 64 positions lie in at most 64 entries from lane 0's on.
    auto advance = [&]() {
        j += FMM_WAVE;
        if (__any(j >= e)) {
            do {
                q += j >= e ? 4 : 0;
                if (__any(q >= 4 * FMM_WAVE)) {
                    const int q0 = __builtin_amdgcn_readfirstlane(q);
                    base += q0 >> 2;
                    q -= q0;
                    fetch();
                }
                e = pick(q, end0);
                sh = pick(q, shift0);
            } while (__any(j >= e));
        }
    };
    int left = t.count;
    while (left > 0) {
        // a loop of its own, so that the sums stay in place
        while (left >= FMM_WAVE && !__any((uint32_t)(j + sh - t.sb) < (uint32_t)t.r)) {
            const auto src = load((uint32_t)(j + sh));
            advance();
            fast(src);
            left -= FMM_WAVE;
        }
        if (left > 0) {
            const uint32_t i = (uint32_t)(j + sh);
            const auto src = load(i);
            const bool on = lane < left;
            advance();
            checked(src, i, on);
            left -= FMM_WAVE;
        }
    }
}

// element i of an array of 32-byte elements (i < 2^31): the address is one
// shift-and-add
__device__ __forceinline__ double4 load32(const double4 *a, uint32_t i) {
    return *reinterpret_cast<const double4 *>(reinterpret_cast<const char *>(a) +
                                              ((uint64_t)(i + i) << 4));
}

// Sum of four values over the wavefront: on return every lane of row 0 (lanes
// 0..15) holds the total of a, row 1 that of c, row 2 that of b, row 3 that of
// d.  Two lane-half swaps and one row swap halve the values before the last
// four steps inside a row.
__device__ __forceinline__ void swap32(double &a, double &b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a),
                                                   (unsigned)__double2loint(b), false, false);
    const u2 hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a),
                                                   (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)hi.x, (int)lo.x);
    b = __hiloint2double((int)hi.y, (int)lo.y);
}
__device__ __forceinline__ void swap16(double &a, double &b) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a),
                                                   (unsigned)__double2loint(b), false, false);
    const u2 hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a),
                                                   (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)hi.x, (int)lo.x);
    b = __hiloint2double((int)hi.y, (int)lo.y);
}
__device__ __forceinline__ double wave_sum4(double a, double b, double c, double d) {
    swap32(a, b);
    swap32(c, d);
    double u = a + b, v = c + d;     // lower half: totals of a / c, upper: of b / d
    swap16(u, v);
    double w = u + v;
    w += dpp_double<DPP_ROW_ROR + 8>(w);
    w += dpp_double<DPP_ROW_ROR + 4>(w);
    w += dpp_double<DPP_ROW_ROR + 2>(w);
    w += dpp_double<DPP_ROW_ROR + 1>(w);
    return w;
}
// component (0..3 for a..d) that wave_sum4 leaves in this lane's row
__device__ __forceinline__ int wave_sum4_component() {
    const int row = lane_id() / 16;
    return ((row & 1) << 1) | (row >> 1);
}

// ---- exact sums over all sources (a slice [j0, j1) per wavefront) -------------
// Sinks of one wavefront: DIRECT_R of them, entries t0.. of the sink list (or
// particles t0.. where the list is null), repeated past the end.  pos[k]: their
// particle indices (scalar registers); *bad is set for an index outside [0, n),
// whose sums are not written.
struct DirectSinks {
    int64_t t0;
    int64_t idx[DIRECT_R];
    unsigned valid;          // bit k: entry t0 + k exists and is in range
};
__device__ __forceinline__ int64_t readlane64(int64_t v, int l) {
    const int lo = __builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint64_t)(uint32_t)lo);
}
__device__ __forceinline__ DirectSinks direct_sinks(int64_t wave, int64_t n, int64_t nsinks,
                                                    const int64_t *sinks, int *bad) {
    DirectSinks d;
    d.t0 = wave * DIRECT_R;
    const int k = lane_id() & (DIRECT_R - 1);
    const int64_t t = d.t0 + k;
    int64_t i = t < nsinks ? (sinks ? sinks[t] : t) : 0;
    const bool ok = t < nsinks && i >= 0 && i < n;
    if (bad && t < nsinks && !ok) atomicOr(bad, 1);
    if (!ok) i = 0;
    d.valid = (unsigned)(__ballot(ok) & ((1u << DIRECT_R) - 1u));
#pragma unroll
    for (int q = 0; q < DIRECT_R; ++q) d.idx[q] = readlane64(i, q);
    return d;
}

// The sources [j0, j1), 64 per step: fast(o) where no sink is among them,
// checked(o, on) elsewhere; o = source - j0 of this lane, on: it exists.
template <class Fast, class Checked>
__device__ __forceinline__ void direct_steps(const DirectSinks &d, int64_t j0, int64_t j1,
                                             Fast &&fast, Checked &&checked) {
    const uint32_t lane = lane_id();
    const uint32_t len = slice_length(j0, j1);       // chunks hold at most 2^31 sources
    uint32_t o = 0;
    while (o < len) {
        // the first sink from here on, if any
        uint32_t next = UINT_MAX;
#pragma unroll
        for (int q = 0; q < DIRECT_R; ++q) {
            const int64_t r = d.idx[q] - j0;
            if (r >= (int64_t)o && r < (int64_t)len) next = min(next, (uint32_t)r);
        }
        const uint32_t stop = min(len, next);
        while (o + FMM_WAVE <= stop) {
            fast(o + lane);
            o += FMM_WAVE;
        }
        if (o < len) {
            checked(o + lane, o + lane < len);
            o += FMM_WAVE;
        }
    }
}

}  // namespace fmm
