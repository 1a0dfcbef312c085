// Device functions shared by the verification kernels (kernels.hip) and the
// self-join kernels (join.hip): wavefront helpers, the required overlap of a
// pair, and the merges.
#pragma once

#include "ssj_device.h"

namespace ssj {
namespace {

// Required overlap of a pair with sizes na, nb under the request's rule
// (paper Table 1, in integers).
//
// Cosine for sizes below kCosineSizes and threshold terms below kCosineTerms:
// the least o with (o den)^2 >= num^2 na nb.  The single-precision estimate of
// num / den sqrt(na nb), below 2^16, is off by less than 2^-5 (five roundings
// of 2^-23 at most), so its integer part less one is at most three below o and
// never above it; exact steps finish the job.  3.4M pairs of two collections of
// short sets at 3/5: 187.5 us a pass with the 128-bit form, 183.5 us so.
__device__ __forceinline__ uint32_t cosine_overlap_small(uint32_t na, uint32_t nb, uint32_t num, uint32_t den,
                                                         float ratio) {
    const uint32_t p = na * nb;
    const unsigned long long x = (unsigned long long)(num * num) * p;
    const uint32_t e = (uint32_t)(ratio * __builtin_amdgcn_sqrtf((float)p));
    uint32_t o = e > 0u ? e - 1u : 0u;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const unsigned long long v = o * den;
        o += v * v < x ? 1u : 0u;
    }
    return o;
}

__device__ __forceinline__ uint32_t cosine_overlap(uint32_t na, uint32_t nb, unsigned long long tn,
                                                   unsigned long long td) {
    // least o with (o td)^2 >= tn^2 na nb; both sides stay below 2^124.  A
    // double estimate lands within one of it and exact steps finish the job.
    const unsigned __int128 x = (unsigned __int128)(tn * tn) * ((unsigned long long)na * nb);
    unsigned long long o = (unsigned long long)ceil((double)tn * sqrt((double)na * (double)nb) / (double)td);
    auto sq = [&](unsigned long long v) { return (unsigned __int128)(v * td) * (v * td); };
    while (o > 0 && sq(o - 1) >= x) --o;
    while (sq(o) < x) ++o;
    return (uint32_t)o;
}

// C: whether the instance handles the Cosine rule (its 128-bit arithmetic
// costs registers in every kernel that contains it, so only launches with a
// Cosine request use such an instance).
template <bool C>
__device__ __forceinline__ uint32_t required_overlap(uint32_t na, uint32_t nb, const Request& R) {
    if constexpr (C) {
        if (R.rule == kCosine) {
            if (R.cosine_ratio != 0.0f)
                return cosine_overlap_small(na, nb, (uint32_t)R.num, (uint32_t)R.den, R.cosine_ratio);
            return cosine_overlap(na, nb, R.num, R.den);
        }
    }
    if (R.rule == kConstant) return (uint32_t)R.num;
    const unsigned long long L = (unsigned long long)na + nb;
    const unsigned long long x = R.num * L + R.den - 1ull;
    if ((x >> 32) == 0ull) {
        // ceil(num L / den) = floor(x / den) by a multiply with the request's
        // precomputed magic number (the round-up method for unsigned division
        // by an invariant integer of Granlund and Montgomery, PLDI 1994)
        const uint32_t n = (uint32_t)x;
        const uint32_t t = __umulhi(R.dmagic, n);
        return (t + ((n - t) >> (R.dshift & 0xffu))) >> (R.dshift >> 8);
    }
    return (uint32_t)(x / R.den);
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

__device__ __forceinline__ unsigned long long ballot(bool p) { return __ballot(p); }

// Value of v held by lane src of the same wavefront.
__device__ __forceinline__ int bperm(int v, int src) {
    return __builtin_amdgcn_ds_bpermute(src << 2, v);
}

// Orders one wavefront's LDS accesses: writes by some lanes before reads by
// others (the LDS serves a wavefront's operations in issue order; the fences
// keep the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Waits until every memory operation of the wavefront has completed.
__device__ __forceinline__ void memory_wait() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// Counters that other workgroups of the launch add to.
__device__ __forceinline__ uint32_t load_agent(const unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_agent(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Number of set bits of m below the calling lane.
__device__ __forceinline__ uint32_t mbcnt(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// One round of the tile merge of G lanes of one wavefront (lanes gbase ..
// gbase+G-1, g = lane - gbase) at merge position (i, j): lane g holds a = A[i+g]
// if g < ka and b = B[j+g] if g < kb.  Each lane finds its a-token in the
// s tile by binary search over the lanes; the side whose tile ends lower is
// consumed whole, the other up to that end, so an equal pair on the seam is
// counted exactly once.  Control flow is uniform inside the group, so the
// cross-lane permutes only read lanes that are active.
template <int G>
__device__ __forceinline__ void group_round(int32_t a, int32_t b, int ka, int kb, int g, int gbase,
                                            uint32_t& i, uint32_t& j, uint32_t& o) {
    const unsigned long long gmask =
        (G == kWave) ? ~0ull : (((1ull << (G % kWave)) - 1ull) << gbase);
    const bool va = g < ka, vb = g < kb;
    const int32_t amax = bperm(a, gbase + ka - 1);
    const int32_t bmax = bperm(b, gbase + kb - 1);
    // pos = number of s-tile tokens below a (capped at G-1)
    int pos = 0;
#pragma unroll
    for (int step = G / 2; step >= 1; step >>= 1) {
        const int k = pos + step - 1;
        const int32_t v = bperm(b, gbase + k);
        if (k < kb && v < a) pos += step;
    }
    const int32_t at = bperm(b, gbase + pos);
    const bool hit = va && pos < kb && at == a;
    const uint32_t nh = (uint32_t)__popcll(ballot(hit) & gmask);
    const uint32_t na_le = (uint32_t)__popcll(ballot(va && a <= bmax) & gmask);
    const uint32_t nb_le = (uint32_t)__popcll(ballot(vb && b <= amax) & gmask);
    // value selects (branches that update i or j by reference end up as a
    // select of addresses, which puts i and j in scratch memory)
    const bool a_low = amax < bmax, b_low = bmax < amax;
    i += b_low ? na_le : (uint32_t)ka;
    j += a_low ? nb_le : (uint32_t)kb;
    o += nh;
}

// Tile merge of G lanes from merge state (i, j, o), loading each tile.
template <int G>
__device__ __forceinline__ bool merge_group(const int32_t* __restrict__ A, uint32_t na,
                                            const int32_t* __restrict__ B, uint32_t nb,
                                            uint32_t alpha, int g, int gbase, uint32_t i = 0,
                                            uint32_t j = 0, uint32_t o = 0) {
    for (;;) {
        if (o >= alpha) return true;
        const uint32_t ra = na - i, rb = nb - j;
        if (o + min(ra, rb) < alpha) return false;
        const int ka = (int)min(ra, (uint32_t)G), kb = (int)min(rb, (uint32_t)G);
        const int32_t a = g < ka ? A[i + g] : 0;
        const int32_t b = g < kb ? B[j + g] : 0;
        group_round<G>(a, b, ka, kb, g, gbase, i, j, o);
    }
}

// The tile merge of G lanes (lanes gbase .. gbase + G - 1, g = lane - gbase)
// with tiles of 4 G tokens, from merge state (i, j, o): four tokens per lane and
// side, so a round consumes four times what one of merge_group<G> does for about
// the same chain of a load, a search and a few counts.  The s tile is searched
// in LDS (sb, 4 G words of the group), padded with the largest value, so the
// search has no bounds.  Control flow is uniform inside the group.  The merges
// that 620,000 pairs of long sets spill, 16 lanes each: kernel 35 -> 21 us.
constexpr uint32_t kWideTile = 4u * kWave;
template <int G>
__device__ __forceinline__ bool merge_wide(const int32_t* __restrict__ A, uint32_t na, const int32_t* __restrict__ B,
                                           uint32_t nb, uint32_t alpha, uint32_t i, uint32_t j, uint32_t o, int g,
                                           int gbase, uint32_t* sb) {
    constexpr uint32_t kTile = 4u * (uint32_t)G;
    const unsigned long long gmask = (G == kWave) ? ~0ull : (((1ull << (G % kWave)) - 1ull) << gbase);
    for (;;) {
        if (o >= alpha) return true;
        const uint32_t ra = na - i, rb = nb - j;
        if (o + min(ra, rb) < alpha) return false;
        const uint32_t ka = min(ra, kTile), kb = min(rb, kTile);
        // (tokens are below 2^31)
        const uint32_t amax = (uint32_t)A[i + ka - 1u], bmax = (uint32_t)B[j + kb - 1u];
        uint32_t a[4], b[4], pos[4];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t x = k * (uint32_t)G + (uint32_t)g;
            a[k] = x < ka ? (uint32_t)A[i + x] : 0xffffffffu;
            b[k] = x < kb ? (uint32_t)B[j + x] : 0xffffffffu;
            pos[k] = 0;
        }
        wave_sync();
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) sb[k * (uint32_t)G + (uint32_t)g] = b[k];
        wave_sync();
#pragma unroll
        for (uint32_t step = kTile / 2u; step >= 1u; step >>= 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) pos[k] += sb[pos[k] + step - 1u] < a[k] ? step : 0u;
        }
        uint32_t nh = 0, na_le = 0, nb_le = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            nh += (uint32_t)__popcll(ballot(sb[pos[k]] == a[k] && a[k] != 0xffffffffu) & gmask);
            na_le += (uint32_t)__popcll(ballot(a[k] <= bmax) & gmask);
            nb_le += (uint32_t)__popcll(ballot(b[k] <= amax) & gmask);
        }
        i += bmax < amax ? na_le : ka;
        j += amax < bmax ? nb_le : kb;
        o += nh;
    }
}

// Lane 0's value of v (all lanes active).
__device__ __forceinline__ unsigned long long lane0_u64(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

// Maximum of v over lanes 0 .. lane of the wavefront (v >= 0): within each
// row of 16 lanes by shifted maxima (DPP row shifts), then across rows from
// the rows' last lanes.
__device__ __forceinline__ uint32_t wave_max_scan(uint32_t v, int lane) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));  // row_shr:8
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
    const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
    const int row = lane >> 4;
    const uint32_t below = row == 0 ? 0u : row == 1 ? r0 : row == 2 ? max(r0, r1) : max(max(r0, r1), r2);
    return max(v, below);
}

// One window step on the current 4-token windows a (set positions ba ..
// ba + 3 of A) and b (bb .. bb + 3 of B), with i and j tokens consumed
// (ba <= i < min(ba + 4, na), the same for j): the window with the lower
// last token is consumed whole, the other up to that token (both on equal
// ones), and o counts the matches among the unconsumed tokens.  Consumed
// tokens are exactly those up to the last consumption point, and slots past
// a set's end hold -1 (the smallest signed, the largest unsigned value), so:
// a window's largest token is the largest of its four slots; an unconsumed
// real token of A is one at a position >= i that is <= bmax as unsigned
// (larger ones cannot match and are not consumed); and such a token can only
// equal an unconsumed token of B, so its matches need no test on b's side.
__device__ __forceinline__ void step_windows(const int32_t (&a)[4], const int32_t (&b)[4], uint32_t ba,
                                             uint32_t bb, uint32_t na, uint32_t nb, uint32_t& i, uint32_t& j,
                                             uint32_t& o) {
    const int32_t amax = max(max(a[0], a[1]), max(a[2], a[3]));
    const int32_t bmax = max(max(b[0], b[1]), max(b[2], b[3]));
    uint32_t hits = 0, na_le = 0, nb_le = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool va = ba + k >= i && (uint32_t)a[k] <= (uint32_t)bmax;
        const bool vb = bb + k >= j && (uint32_t)b[k] <= (uint32_t)amax;
        bool hit = false;
#pragma unroll
        for (int t = 0; t < 4; ++t) hit |= a[k] == b[t];
        hits += (va && hit) ? 1u : 0u;
        na_le += va ? 1u : 0u;
        nb_le += vb ? 1u : 0u;
    }
    i = bmax < amax ? i + na_le : min(ba + 4u, na);
    j = amax < bmax ? j + nb_le : min(bb + 4u, nb);
    o += hits;
}

// One lane's merge continued from state (i, j, o) over 16-byte windows of
// the two token lists (A from slot sa of tok_a, B from slot sb of tok_b;
// every set starts on a 16-byte boundary of its token array): window w of a
// side holds its tokens 4w .. 4w+3.  A step merges the
// unconsumed tokens of the current windows of both sides (up to 4 x 4
// comparisons) and consumes, as in the tile merge, every token that can have
// no partner beyond the two windows: all of the window with the lower end,
// and the tokens of the other window up to that end (both windows when the
// ends are equal).  The window after the current one of each side is always
// one step in flight: a step takes it over where the current window is used
// up, and then requests the next one unconditionally (a side that did not
// advance requests the window it already holds, a cache hit; a conditional
// load ends up in a temporary register plus a copy that waits for it).  The
// scheduling barrier keeps those loads after the selects that read the
// registers they refill, for the same reason.  The pair must be undecided at (i, j, o), so
// i < na and j < nb; (i, j, o) hold the state where the merge stopped.  After
// budget steps a merge still undecided stops with *spilled set (all lanes
// enter together, so the step count is the same in every lane and the cut is
// a wave-uniform branch).
//
// The windows as separate 32-bit values (selects on whole vectors become
// address selects into scratch memory): the current and the next one of each
// side.
struct Windows {
    int32_t a[4], b[4], an[4], bn[4];
};

__device__ __forceinline__ void unpack_window(uint4 v, int32_t (&d)[4]) {
    d[0] = (int32_t)v.x;
    d[1] = (int32_t)v.y;
    d[2] = (int32_t)v.z;
    d[3] = (int32_t)v.w;
}

// The windows at merge state (i, j), i < na and j < nb.
__device__ __forceinline__ void load_windows(const int32_t* __restrict__ tok_a, uint32_t sa, uint32_t na,
                                             const int32_t* __restrict__ tok_b, uint32_t sb, uint32_t nb, uint32_t i,
                                             uint32_t j, Windows& w) {
    const uint4* __restrict__ t4a = reinterpret_cast<const uint4*>(tok_a);
    const uint4* __restrict__ t4b = reinterpret_cast<const uint4*>(tok_b);
    const uint32_t qa = sa >> 2, qb = sb >> 2;              // first window of each set
    const uint32_t la = (na - 1u) >> 2, lb = (nb - 1u) >> 2;  // last window index
    unpack_window(t4a[qa + (i >> 2)], w.a);
    unpack_window(t4b[qb + (j >> 2)], w.b);
    unpack_window(t4a[qa + min((i >> 2) + 1u, la)], w.an);
    unpack_window(t4b[qb + min((j >> 2) + 1u, lb)], w.bn);
}

__device__ __forceinline__ bool merge_loaded(const int32_t* __restrict__ tok_a, uint32_t sa,
                                             uint32_t na, const int32_t* __restrict__ tok_b,
                                             uint32_t sb, uint32_t nb, uint32_t alpha, uint32_t& i,
                                             uint32_t& j, uint32_t& o, uint32_t budget, bool* spilled, Windows& w) {
    const uint4* __restrict__ t4a = reinterpret_cast<const uint4*>(tok_a);
    const uint4* __restrict__ t4b = reinterpret_cast<const uint4*>(tok_b);
    const uint32_t qa = sa >> 2, qb = sb >> 2;
    const uint32_t la = (na - 1u) >> 2, lb = (nb - 1u) >> 2;
    uint32_t wa = i >> 2, wb = j >> 2;
    for (uint32_t step = 1;; ++step) {
        const uint32_t ba = wa << 2, bb = wb << 2;
        step_windows(w.a, w.b, ba, bb, na, nb, i, j, o);
        if (o >= alpha) return true;
        if (o + min(na - i, nb - j) < alpha) return false;
        if (step >= budget) {
            *spilled = true;
            return false;
        }
        const bool adv_a = i >= ba + 4u, adv_b = j >= bb + 4u;
        wa += adv_a ? 1u : 0u;
        wb += adv_b ? 1u : 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            w.a[k] = adv_a ? w.an[k] : w.a[k];
            w.b[k] = adv_b ? w.bn[k] : w.b[k];
        }
        __builtin_amdgcn_sched_barrier(0);
        unpack_window(t4a[qa + min(wa + 1u, la)], w.an);
        unpack_window(t4b[qb + min(wb + 1u, lb)], w.bn);
    }
}

__device__ __forceinline__ bool merge_windows(const int32_t* __restrict__ tok_a, uint32_t sa,
                                              uint32_t na, const int32_t* __restrict__ tok_b,
                                              uint32_t sb, uint32_t nb, uint32_t alpha, uint32_t& i,
                                              uint32_t& j, uint32_t& o, uint32_t budget, bool* spilled) {
    Windows w;
    load_windows(tok_a, sa, na, tok_b, sb, nb, i, j, w);
    return merge_loaded(tok_a, sa, na, tok_b, sb, nb, alpha, i, j, o, budget, spilled, w);
}

}  // namespace
}  // namespace ssj
