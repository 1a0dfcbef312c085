// Verification kernels for gfx950 (CDNA4, wave64).
//
// A candidate pair (r, s) is similar iff its overlap o = |r & s| reaches the
// required overlap alpha of its similarity function (paper Sec. 3, Definition
// 1; the equivalent overlaps of Table 1 in integers): for Jaccard
//     alpha = ceil(t_num * (|r| + |s|) / (t_num + t_den)),
// for Dice ceil(t_num (|r| + |s|) / (2 t_den)), for Cosine the least o with
// o^2 t_den^2 >= t_num^2 |r| |s|, for Overlap ceil(t_num / t_den).  The r side
// of a pair reads one collection, the s side another in an R-S join (the same
// one in a self-join).
// The overlap is found by walking the two sorted token lists and stopping as
// soon as o >= alpha (accept) or o + min(tokens left in r, tokens left in s)
// < alpha (reject: alpha is out of reach) -- the early-terminating merge of
// paper Sec. 3.1.  Any sound stopping rule yields the same decisions.
//
// Mappings of pairs onto lanes (the paper's alternatives A/B/C of Sec. 3.3.2
// give a probe set to a thread or a block; here the unit is one pair):
//   * one thread per pair: an upper bound of the overlap from two bitmaps of
//     token hashes (signatures), which rejects nearly all pairs that are not
//     similar; for the others the merge of the first six tokens of both sets,
//     kept in their 32-byte set records, in straight-line code, then, for a
//     pair still undecided, a merge over 16-byte windows of the token arrays
//     (every set starts on a 16-byte boundary) with the next window in
//     flight; optionally cut off after a budget of window steps, the pair
//     then being queued for the second kernel;
//   * a group of G lanes (G = 4..64) of one wavefront per pair: tile merge;
//   * a wavefront per pair with tiles of 256 tokens, the s tile in LDS.
// The tile merge advances in rounds.  A round loads the next G tokens of r
// (one per lane) and of s, counts the r tokens found in the s tile by a
// binary search over the tile (cross-lane permutes or LDS), and then
// consumes every token that can have no partner beyond the two tiles: if
// max(r tile) < max(s tile) the whole r tile plus the s tokens <= max(r tile)
// are consumed (and symmetrically; both tiles when the maxima are equal).
// Every equal pair of tokens lies in the consumed part of both sides in the
// round that finds it and in no later round, so each match is counted
// exactly once; the stopping rule is checked before every round.
//
// Scheduling.  One launch carries up to kMaxReq requests (candidate arrays
// with their own threshold and output).  In the in-order kernel every
// wavefront walks chunks of kWave consecutive pairs of one request (a static
// grid-stride split: with early termination the cost of a pair depends on its
// first few tokens, not on its length, so in-order chunks are balanced), with
// the loads of the next chunks in flight.  Optionally, pairs whose length
// class |r| + |s| is at or above defer_from are not verified there but queued
// per class (collected in LDS, one global atomic per flush); a second,
// persistent kernel drains those queues with the class's own mapping, each by
// a static split.
// Passing pairs are compacted in LDS (a ballot of the pass flags and each
// lane's rank among the passing lanes) and moved to the request's output
// with one global atomic per flush.  The in-order kernel keeps all of this
// per wavefront, so it has no workgroup barrier; with a group per pair, and where
// shares are long, each wavefront lowers its priority as it works through its
// share, so that the youngest wavefronts of a SIMD do not finish long after the
// rest.
#include <algorithm>
#include <cstddef>

#include "merge_device.h"
#include "ssj_device.h"

namespace ssj {
namespace {

// Requests the kernel's arguments (up to the first request's) at its beginning, a
// word of every cache line side by side: they lie in host memory, and lines that
// are first asked for along the way are waited for one after the other (2,000
// pairs under a plan with two kernels 21.3 -> 20.4 us).
__device__ __forceinline__ void touch_args() {
    auto k = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x = 0;
#pragma unroll
    for (uint32_t o = 0; o < (uint32_t)(offsetof(LaunchArgs, req) + sizeof(Request)) / 4u; o += 16u) x |= k[o];
    asm volatile("" ::"s"(x));
}

// Set record: {start, len, first kHeadTokens tokens} in two 16-byte words
// (slots past the end of a shorter set hold -1).
__device__ __forceinline__ uint2 set_desc(const LaunchArgs& a, int id) {
    const uint4 v = a.heads[2 * id];
    return make_uint2(v.x, v.y);
}

// The same for a set of the s-side collection.
__device__ __forceinline__ uint2 set_desc_s(const LaunchArgs& a, int id) {
    const uint4 v = a.heads_s[2 * id];
    return make_uint2(v.x, v.y);
}

// Candidate pair k of a request.
__device__ __forceinline__ int2 load_pair(const int2* __restrict__ cand, uint32_t k) {
    return cand[k];
}

// One thread: sequential early-terminating merge.
__device__ __forceinline__ bool merge_thread(const int32_t* __restrict__ A, uint32_t na,
                                             const int32_t* __restrict__ B, uint32_t nb,
                                             uint32_t alpha) {
    uint32_t i = 0, j = 0, o = 0;
    for (;;) {
        if (o >= alpha) return true;
        const uint32_t rem = min(na - i, nb - j);
        if (o + rem < alpha) return false;
        const int32_t x = A[i], y = B[j];
        i += (x <= y);
        j += (y <= x);
        o += (x == y);
    }
}

// The same merge from the start, with the first tiles already loaded by the
// caller: a0 = A[min(g, na-1)], b0 = B[min(g, nb-1)] (a software pipeline
// issues them one pair ahead, so a pair decided within its first tiles waits
// for no load).
template <int G>
__device__ __forceinline__ bool merge_group_first(const int32_t* __restrict__ A, uint32_t na,
                                                  const int32_t* __restrict__ B, uint32_t nb,
                                                  uint32_t alpha, int g, int gbase, int32_t a0,
                                                  int32_t b0) {
    if (alpha == 0u) return true;
    if (min(na, nb) < alpha) return false;
    const int ka = (int)min(na, (uint32_t)G), kb = (int)min(nb, (uint32_t)G);
    uint32_t i = 0, j = 0, o = 0;
    group_round<G>(g < ka ? a0 : 0, g < kb ? b0 : 0, ka, kb, g, gbase, i, j, o);
    return merge_group<G>(A, na, B, nb, alpha, g, gbase, i, j, o);
}

// Token min(g, n-1) of a set with descriptor d = (start, n), n >= 1: the
// lane's token of the set's first tile (clamped, so the load is unconditional).
__device__ __forceinline__ int32_t first_tile_token(const int32_t* __restrict__ tok, uint2 d, int g) {
    return tok[d.x + min((uint32_t)g, d.y - 1u)];
}

// Whether r indexes the r-side collection and s the s-side one.
__device__ __forceinline__ bool ids_ok(int2 pr, const LaunchArgs& a) {
    return (uint32_t)pr.x < a.n_sets && (uint32_t)pr.y < a.n_sets_s;
}

__device__ __forceinline__ int class_of(uint32_t L, const LaunchArgs& a) {
    int cls = kClasses - 1;
#pragma unroll
    for (int q = kClasses - 2; q >= 0; --q)
        if (L <= a.bounds[q]) cls = q;
    return cls;
}

// Request holding global pair index gi (prefix sums in pair_off).
__device__ __forceinline__ int request_of_pair(uint32_t gi, const LaunchArgs& a) {
    int r = 0;
    for (int q = 1; q < a.n_req; ++q) r += (gi >= a.pair_off[q]) ? 1 : 0;
    return r;
}

// ---------------------------------------------------------------------------
// Wavefront-private buffers of the in-order kernel.  Every wavefront works on
// its own chunks of kWave consecutive pairs and keeps its own LDS buffers
// (staged output pairs, deferred pairs, hard pairs).  Their fill counts are
// wave-uniform values held in registers, so the kernel needs no workgroup
// barrier: a wavefront slowed by a long merge holds up no other.


// Appends the pairs of the lanes with pass set to the wavefront's staged
// output (ocnt entries so far, wave-uniform).  A request without an output
// buffer only counts.
__device__ __forceinline__ void stage_pass(bool pass, int2 pr, int2* w_out, uint32_t& ocnt,
                                           bool count_only) {
    const unsigned long long m = ballot(pass);
    if (!count_only && pass) w_out[ocnt + mbcnt(m)] = pr;
    ocnt += (uint32_t)__popcll(m);
}

// A launch of few workgroups whose only kernel is the in-order one counts its
// workgroups and its errors in the words of the requests' passing pairs: each
// workgroup ends with one atomic per request, side by side, whose result tells
// the last one that request's count, where otherwise it waits for its counts to
// arrive, for its number among the finished and for the counts again.  (Bits
// 0-39: pairs, 40-55: workgroups, 56-63: workgroups that met an error.)
// 500 candidates in two requests 14.0 -> 13.2 us, 2,000 candidates of one
// 10.9 -> 10.3, 17,000 in four 18.0 -> 16.7.
constexpr uint32_t kQuickGrid = 128;
constexpr int kDoneShift = 40, kErrShift = 56;
constexpr unsigned long long kCountMask = (1ull << kDoneShift) - 1ull;
template <bool GR>
__device__ __forceinline__ bool quick_end(const LaunchArgs& a) {
    // (a pre-pass of a grouped launch leaves its errors in memory)
    return a.two_kernels == 0u && gridDim.x <= kQuickGrid && (!GR || a.chunk_g == nullptr);
}

// Moves the wavefront's c staged pairs of request r to the request's output
// with one global atomic.  The pairs of a request without an output buffer are
// only counted, in the workgroup's LDS (s_only).  Called by the whole
// wavefront.
__device__ void wave_flush_out(const LaunchArgs& a, int r, uint32_t c, const int2* w_out, uint32_t* s_only) {
    const int lane = lane_id();
    if (a.req[r].cap == 0) {
        if (lane == 0) atomicAdd(&s_only[r], c);
        return;
    }
    wave_sync();
    unsigned long long base = 0ull;
    if (lane == 0) base = atomicAdd(&a.ctr->out_count[r], (unsigned long long)c);
    base = lane0_u64(base) & kCountMask;
    const Request& R = a.req[r];
    for (uint32_t i = (uint32_t)lane; i < c; i += kWave) {
        const unsigned long long k = base + i;
        if (k < R.cap) R.out[k] = w_out[i];
    }
    wave_sync();
}

// Called by one wavefront of every workgroup when all memory operations of
// the workgroup have completed (memory_wait in each of its wavefronts): the
// workgroup counts as finished, on one of kSlots addresses, and the last one of
// the grid publishes each request's count (-1 after an id error) and returns
// the counters to zero for the next launch.  Counts and flags are read with
// atomics, which the others' completed atomics precede, so no fence is needed
// (a device-scope fence per workgroup writes back the XCD's L2 and cost about
// 60 us per launch; a kernel of its own for this took 4.6 us).
__device__ void finish_workgroup(const LaunchArgs& a) {
    const int lane = lane_id();
    uint32_t last = 0;
    if (lane == 0) {
        // (a small grid needs no slots, a single workgroup no count: each
        // step is an atomic's latency at the end of the launch)
        const uint32_t slot = blockIdx.x % kSlots;
        const uint32_t of = (gridDim.x - slot + kSlots - 1u) / kSlots;
        if (gridDim.x == 1u)
            last = 1u;
        else if (gridDim.x <= kSlots || atomicAdd(&a.ctr->slot[slot].done, 1u) == of - 1u)
            last = atomicAdd(&a.ctr->done, 1u) == min(gridDim.x, kSlots) - 1u ? 1u : 0u;
    }
    if (__builtin_amdgcn_readfirstlane((int)last) == 0) return;
    if (lane < a.n_req) {
        const unsigned long long cnt = load_agent(&a.ctr->out_count[lane]);
        const unsigned err = load_agent(&a.ctr->err[lane]);
        *a.req[lane].d_count = err ? -1ll : (long long)cnt;
        a.ctr->out_count[lane] = 0ull;
        a.ctr->err[lane] = 0u;
    }
    if (lane < kQueues) {
        a.ctr->tail[lane] = 0u;
    }
    if (lane < (int)kSlots) {
        a.ctr->slot[lane].done = 0u;
        a.ctr->slot[lane].many = 0u;
    }
    if (lane == 0) a.ctr->done = 0u;
}

// Entries of class q in the wavefront's deferred queues: 8 bits per class
// in one wave-uniform word (a queue never holds more than defer_cap <= 255).
__device__ __forceinline__ uint32_t dcount(unsigned long long dc, int q) {
    return (uint32_t)(dc >> (8 * q)) & 0xffu;
}

// Appends the pairs (global pair index gi) of the lanes with mine set to
// the wavefront's LDS queue q.
__device__ __forceinline__ void queue_lanes(const LaunchArgs& a, bool mine, int q, uint32_t gi,
                                            uint32_t* w_defer, unsigned long long& dc) {
    const unsigned long long m = ballot(mine);
    if (mine) w_defer[(uint32_t)(q - a.defer_from) * a.defer_cap + dcount(dc, q) + mbcnt(m)] = gi;
    dc += (unsigned long long)__popcll(m) << (8 * q);
}

// Queues deferred pairs in the wavefront's LDS queue of their class, and
// spilled merges in its spill queue (after the class queues).
__device__ __forceinline__ void defer_pass(const LaunchArgs& a, bool defer, int cls, bool spill,
                                           uint32_t gi, uint32_t* w_defer, unsigned long long& dc) {
    for (int q = a.defer_from; q < kClasses; ++q) queue_lanes(a, defer && cls == q, q, gi, w_defer, dc);
    if (spilling(a)) queue_lanes(a, spill, kSpillQ, gi, w_defer, dc);
}

// One past the last LDS queue of the in-order kernel's wavefronts.
__device__ __forceinline__ int queue_end(const LaunchArgs& a) {
    return spilling(a) ? kQueues : kClasses;
}

// Moves the wavefront's c queued pairs of class q to the global queue.
__device__ void wave_flush_deferred(const LaunchArgs& a, int q, uint32_t c, const uint32_t* w_defer) {
    wave_sync();
    const int lane = lane_id();
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(&a.ctr->tail[q], c);
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    const uint32_t* src = w_defer + (uint32_t)(q - a.defer_from) * a.defer_cap;
    uint32_t* dst = a.queues + (size_t)q * a.qcap + base;
    for (uint32_t i = (uint32_t)lane; i < c; i += kWave) dst[i] = src[i];
    wave_sync();
}

// Wavefront priority from progress: 3 before the first quarter of its
// chunks is done, down to 0 in the last quarter.  The SIMD's arbiter favours
// the oldest wavefronts among those of equal priority, so with equal shares
// of chunks the youngest ones would otherwise finish long after the rest and
// leave the end of the launch to a few wavefronts; a wavefront that is ahead
// now yields to one that is behind.  quarter[k - 1] = ceil(k share / 4) for
// k = 1, 2, 3 (share: the wavefront's chunk count), so that done chunks are
// past the k-th quarter when done >= quarter[k - 1], without a division per
// chunk.  done, quarter and level are wave-uniform.
__device__ __forceinline__ void progress_priority(uint32_t done, const uint32_t (&quarter)[3], uint32_t& level) {
    const uint32_t l = 3u - (done >= quarter[0] ? 1u : 0u) - (done >= quarter[1] ? 1u : 0u) -
                       (done >= quarter[2] ? 1u : 0u);
    if (l == level) return;
    level = l;
    switch (l) {
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
    }
}

// Request and first pair index of chunk T (prefix sums in tile_off, in
// chunks of kWave pairs).
__device__ __forceinline__ void chunk_origin(const LaunchArgs& a, uint32_t T, int* r, uint32_t* kb) {
    if (a.n_req == 1) {  // the common launch of one request: no search
        *r = 0;
        *kb = T * (uint32_t)kWave;
        return;
    }
    int q = 0;
    while (q + 1 < a.n_req && a.tile_off[q + 1] <= T) ++q;
    *r = q;
    *kb = (T - a.tile_off[q]) * (uint32_t)kWave;
}

// ---------------------------------------------------------------------------
// Candidates of a chunk of a flat or a grouped request.  Loading and finding
// the pair are separate steps, so that a pipeline can issue a chunk's loads
// one iteration before it needs its pairs.  A grouped chunk's lanes load
// their s ids and a window of 64 consecutive groups from the chunk's first
// group (chunk_g); each lane then finds its group among them.

// The loads of a lane's candidate: the pair (flat), or the s id in p.y and
// the lane's entry of the chunk's group window, groups[g0 + lane] (clamped
// to the last group), in gw (grouped).
struct CandLoad {
    int2 p;
    int2 gw;
    uint32_t g0;  // the window's first group (wave-uniform)
};

__device__ __forceinline__ int32_t group_end(const int2* groups, uint32_t g) {
    return reinterpret_cast<const int32_t*>(groups)[2u * g + 1u];
}

// Group x of all requests of the launch (requests located by the prefix sums
// group_off): checks its end against its predecessor's and the request's size,
// and calls write(r, t, g) for every chunk start t * kWave inside its
// candidates.  With ends that do not decrease, end above n or a last end other
// than n, the request's error flag is set and error(r) called; only chunks of the request are ever
// written.
template <class Write, class Error>
__device__ __forceinline__ void group_chunks(const LaunchArgs& a, uint32_t x, Write write, Error error) {
    int r = 0;
    for (int q = 1; q < a.n_req; ++q) r += (x >= a.group_off[q]) ? 1 : 0;
    const Request& R = a.req[r];
    const uint32_t g = x - a.group_off[r];
    const int32_t e = group_end(R.groups, g);
    const int32_t pv = g > 0u ? group_end(R.groups, g - 1u) : 0;
    if (e < pv || (uint32_t)e > R.n || (g + 1u == R.n_groups && (uint32_t)e != R.n)) {
        atomicOr(&a.ctr->err[r], 1u);
        error(r);
        return;
    }
    // 0 <= max(pv, 0) <= e <= n: every t written is below the request's chunk count
    const uint32_t lo = (uint32_t)max(pv, 0), hi = (uint32_t)e;
    for (uint32_t t = (lo + (uint32_t)kWave - 1u) / (uint32_t)kWave; t * (uint32_t)kWave < hi; ++t) write(r, t, g);
}

// First group of chunk c: from the pre-pass, or without one from LDS.
__device__ __forceinline__ uint32_t first_group(const LaunchArgs& a, uint32_t c, const uint32_t* s_chunk) {
    return a.chunk_g != nullptr ? a.chunk_g[c] : s_chunk[c];
}

// First groups of a wavefront's upcoming chunks, one per lane: lane L holds
// chunk_g of the wavefront's chunk with ordinal base + L (its chunk
// first + (base + L) * nw, clamped to the last chunk as the pipelines clamp
// their chunks), so that a grouped chunk's first group is in a register
// before its loads are issued (one vector load per 64 chunks of a wavefront).
template <bool GR>
__device__ __forceinline__ uint32_t load_chunk_groups(const LaunchArgs& a, uint32_t first, uint32_t nw,
                                                      uint32_t n_chunks, uint32_t base, int lane,
                                                      const uint32_t* s_chunk) {
    if constexpr (!GR) return 0u;
    const unsigned long long c = (unsigned long long)first + (unsigned long long)(base + (uint32_t)lane) * nw;
    return first_group(a, c < n_chunks ? (uint32_t)c : n_chunks - 1u, s_chunk);
}

// Issues the loads of the lane's candidate of the chunk at candidate kb of
// request R, whose first group is g0 (chunk_g; unused for a flat request).
// chunk_g entries of a request with malformed groups may be stale (that
// request reports an error): g0 is clamped, so every load stays inside the
// request's buffers.
template <bool GR>
__device__ __forceinline__ CandLoad issue_cand(const LaunchArgs& a, const Request& R, uint32_t kb, int lane,
                                               uint32_t g0) {
    CandLoad c;
    const uint32_t k = kb + (uint32_t)lane;
    const uint32_t kc = k < R.n ? k : R.n - 1u;
    if constexpr (!GR) {
        c.p = load_pair(R.cand, kc);
        c.gw = make_int2(0, 0);
        c.g0 = 0u;
        return c;
    }
    c.g0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(g0, R.n_groups));
    c.p = make_int2(0, R.sids[kc]);
    c.gw = R.n_groups != 0u ? R.groups[min(c.g0 + (uint32_t)lane, R.n_groups - 1u)] : make_int2(-1, -1);
    return c;
}

// The lane's pair from its loads (all lanes of the wavefront call it
// together: cross-lane operations); marks is the wavefront's 64-word LDS
// scratch.  The group of candidate kb + k is the first one whose end exceeds
// it, so its index in a window of ends that do not decrease is the number of
// window groups ending at or before kb + k.  Each window group marks the
// chunk position its end falls on (the largest group index + 1 per
// position, by an LDS maximum), and a running maximum over the positions
// gives every lane that number at once.  A lane past all 64 ends searches
// the next window; a candidate no group covers gets probe id -1 (an id
// error).
template <bool GR>
__device__ __forceinline__ int2 resolve_cand(const LaunchArgs& a, const Request& R, uint32_t kb, int lane,
                                             const CandLoad& c, uint32_t* marks) {
    if constexpr (!GR) return c.p;
    const uint32_t k = kb + (uint32_t)lane;
    const bool valid = k < R.n;
    uint32_t w0 = c.g0;
    int2 e = c.gw;
    int32_t probe = -1;
    bool found = false;
    while (w0 < R.n_groups) {
        const uint32_t ek = w0 + (uint32_t)lane < R.n_groups ? (uint32_t)e.y : 0xffffffffu;
        // chunk candidates before the end of the lane's window group (0 .. 64)
        const uint32_t cpos = ek <= kb ? 0u : min(ek - kb, (uint32_t)kWave);
        marks[lane] = 0u;
        wave_sync();
        if (cpos < (uint32_t)kWave) atomicMax(&marks[cpos], (uint32_t)lane + 1u);
        wave_sync();
        const uint32_t cnt = wave_max_scan(marks[lane], lane);
        wave_sync();  // the marks are cleared again by the next use
        const int32_t pp = bperm(e.x, (int)min(cnt, (uint32_t)kWave - 1u));
        if (!found && cnt < (uint32_t)kWave && w0 + cnt < R.n_groups) {
            probe = pp;
            found = true;
        }
        if (ballot(valid && !found) == 0ull) break;
        w0 += (uint32_t)kWave;
        if (w0 < R.n_groups) e = R.groups[min(w0 + (uint32_t)lane, R.n_groups - 1u)];
    }
    return make_int2(probe, c.p.y);
}

// A queued pair (global pair index gi of request r) in the deferred kernel:
// from the request's pairs, or for a grouped launch its s id and the probe id
// that the in-order kernel stored when it queued the pair.
template <bool GR>
__device__ __forceinline__ int2 queued_pair(const LaunchArgs& a, const Request* reqs, uint32_t gi, int r) {
    const Request& R = reqs[r];
    const uint32_t k = gi - a.pair_off[r];
    if constexpr (GR) return make_int2((int32_t)a.probes[gi], R.sids[k]);
    return load_pair(R.cand, k);
}

// Records the probe id of a pair that the in-order kernel queues (grouped
// launches only; the deferred kernel reads it back by global pair index).
template <bool GR>
__device__ __forceinline__ void note_queued(const LaunchArgs& a, bool queued, int2 pr, uint32_t gi) {
    if constexpr (GR) {
        if (queued) a.probes[gi] = (uint32_t)pr.x;
    }
}

// Set records of a lane's pair: four 16-byte loads (first and second word of
// both sides), issued back to back.  A pair with an invalid id reads record 0
// and is ignored later.
struct LaneRecords {
    uint4 ra0, ra1, rb0, rb1;
};

__device__ __forceinline__ void issue_records(const LaunchArgs& a, int2 pr, LaneRecords& rec) {
    const bool ok = ids_ok(pr, a);
    const int ir = ok ? pr.x : 0, is = ok ? pr.y : 0;
    rec.ra0 = a.heads[2 * ir];
    rec.ra1 = a.heads[2 * ir + 1];
    rec.rb0 = a.heads_s[2 * is];
    rec.rb1 = a.heads_s[2 * is + 1];
}

// Signatures of a lane's pair.
template <int U>
struct Signatures {
    uint4 r[U], s[U];
};

// (ids past the last set read the last one's, with last 0 everything reads
// the first one's)
template <int U>
__device__ __forceinline__ void issue_signatures(const uint4* sig, const uint4* sig_s, uint32_t last_r, uint32_t last_s,
                                                 int2 pr, Signatures<U>& q) {
    const size_t ir = min((uint32_t)pr.x, last_r), is = min((uint32_t)pr.y, last_s);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        q.r[u] = sig[ir * U + u];
        q.s[u] = sig_s[is * U + u];
    }
}

// The most tokens that two sets can share by their signatures.  A token of
// both sets has its bit in both bitmaps, so a set's bits that the other one
// lacks stand for as many tokens of its own: |r| minus those of r, and |s|
// minus those of s, bound the overlap.
template <int U>
__device__ __forceinline__ uint32_t most_shared(const Signatures<U>& q) {
    uint32_t c = 0, nr = 0, ns = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (u > 0) {
            c += (uint32_t)__popc(q.r[u].x & q.s[u].x);
            nr += (uint32_t)__popc(q.r[u].x);
            ns += (uint32_t)__popc(q.s[u].x);
        }
        c += (uint32_t)(__popc(q.r[u].y & q.s[u].y) + __popc(q.r[u].z & q.s[u].z) + __popc(q.r[u].w & q.s[u].w));
        nr += (uint32_t)(__popc(q.r[u].y) + __popc(q.r[u].z) + __popc(q.r[u].w));
        ns += (uint32_t)(__popc(q.s[u].y) + __popc(q.s[u].z) + __popc(q.s[u].w));
    }
    return c + min(q.r[0].x - nr, q.s[0].x - ns);
}

// Merge state after the first tile of one side is consumed, with the first
// H record tokens of each side as the tiles (the tile merge of merge_group,
// done by one lane in straight-line code): with m the smaller of the two
// tile ends, the merge has consumed every token <= m of both tiles, and the
// overlap so far is the number of equal tokens in the two tiles (all of them
// are <= m).  Record slots past the end of a set hold -1; tokens are >= 0, so
// unsigned comparisons with m >= 0 leave those slots out of both counts (sets
// are not empty, so m >= 0).  A larger H gives a state at least as far along
// the same merge.
template <int H>
__device__ __forceinline__ void head_tiles(const int32_t (&A)[H], const int32_t (&B)[H], uint32_t* i,
                                           uint32_t* j, uint32_t* o) {
    int32_t am = A[0], bm = B[0];
#pragma unroll
    for (int x = 1; x < H; ++x) {
        am = max(am, A[x]);
        bm = max(bm, B[x]);
    }
    const uint32_t m = (uint32_t)min(am, bm);
    uint32_t ci = 0, cj = 0, co = 0;
#pragma unroll
    for (int x = 0; x < H; ++x) {
        ci += ((uint32_t)A[x] <= m) ? 1u : 0u;
        cj += ((uint32_t)B[x] <= m) ? 1u : 0u;
        bool hit = false;
#pragma unroll
        for (int y = 0; y < H; ++y) hit |= A[x] == B[y];
        co += (hit && A[x] >= 0) ? 1u : 0u;
    }
    *i = ci;
    *j = cj;
    *o = co;
}

// One window step of the tile merge on the current 4-token windows va (of
// the r side, tokens 4*(i/4).. of a set of na tokens) and vb (s side): the
// side whose window ends lower is consumed whole, the other up to that end
// (both on equal ends); equal tokens inside the unconsumed parts are matches.
// Same rule as the steps of merge_windows.
__device__ __forceinline__ void window_step(uint4 va, uint4 vb, uint32_t na, uint32_t nb, uint32_t& i,
                                            uint32_t& j, uint32_t& o) {
    const int32_t a[4] = {(int32_t)va.x, (int32_t)va.y, (int32_t)va.z, (int32_t)va.w};
    const int32_t b[4] = {(int32_t)vb.x, (int32_t)vb.y, (int32_t)vb.z, (int32_t)vb.w};
    step_windows(a, b, i & ~3u, j & ~3u, na, nb, i, j, o);
}

// Entries of the wavefront's window ring (merge_ring): three 16-byte slots per
// side and lane, slot s of side d of lane l at ring[(3 d + s) * kWave + l]
// (so that a wavefront's accesses to one slot are consecutive).
constexpr uint32_t kRingSlots = 6u * (uint32_t)kWave;

// The merge of merge_windows (same steps, same step budget) with the loads
// two steps ahead instead of one.  Each side's windows pass through a ring of
// three LDS slots of the lane (window w in slot w % 3).  After every step the
// lane requests the window two past its new current one of each side into
// one of two register sets, which is written to the ring two steps later; a
// step reads its two windows from the ring.  The current window of a side
// moves by at most one per step, so every window a step can need has been
// written, and no written window is still needed when its slot is reused; a
// load has two steps to arrive before anything waits for it.  Windows past a
// set's last one are loaded clamped (and never read).
__device__ __forceinline__ bool merge_ring(const int32_t* __restrict__ tok_a, uint32_t sa, uint32_t na,
                                           const int32_t* __restrict__ tok_b, uint32_t sb, uint32_t nb,
                                           uint32_t alpha, uint32_t& i, uint32_t& j, uint32_t& o, uint32_t budget,
                                           bool* spilled, uint4* ring, int lane) {
    const uint4* __restrict__ t4a = reinterpret_cast<const uint4*>(tok_a);
    const uint4* __restrict__ t4b = reinterpret_cast<const uint4*>(tok_b);
    const uint32_t qa = sa >> 2, qb = sb >> 2;              // first window of each set
    const uint32_t la = (na - 1u) >> 2, lb = (nb - 1u) >> 2;  // last window index
    uint4* ra = ring + lane;
    uint4* rb = ring + 3 * kWave + lane;
    auto slot = [](uint32_t w) { return (w % 3u) * (uint32_t)kWave; };
    uint32_t wa = i >> 2, wb = j >> 2;
    ra[slot(wa)] = t4a[qa + wa];
    ra[slot(wa + 1u)] = t4a[qa + min(wa + 1u, la)];
    rb[slot(wb)] = t4b[qb + wb];
    rb[slot(wb + 1u)] = t4b[qb + min(wb + 1u, lb)];
    // set x: the windows two past the first step's (written before step 3)
    uint32_t xwa = wa + 2u, xwb = wb + 2u;
    uint4 xa = t4a[qa + min(xwa, la)], xb = t4b[qb + min(xwb, lb)];
    uint32_t ywa, ywb;
    uint4 ya, yb;
    uint32_t step = 0;
    // one step on the ring: 0 undecided, 1 similar, 2 not similar, 3 cut off
    auto merge_step = [&]() -> int {
        ++step;
        wave_sync();
        const uint4 va = ra[slot(i >> 2)], vb = rb[slot(j >> 2)];
        window_step(va, vb, na, nb, i, j, o);
        if (o >= alpha) return 1;
        if (o + min(na - i, nb - j) < alpha) return 2;
        if (step >= budget) return 3;
        return 0;
    };
    auto finish = [&](int st) {
        if (st == 3) *spilled = true;
        return st == 1;
    };
    int st = merge_step();
    if (st != 0) return finish(st);
    ywa = (i >> 2) + 2u;
    ywb = (j >> 2) + 2u;
    ya = t4a[qa + min(ywa, la)];
    yb = t4b[qb + min(ywb, lb)];
    st = merge_step();
    if (st != 0) return finish(st);
    for (;;) {
        ra[slot(xwa)] = xa;
        rb[slot(xwb)] = xb;
        xwa = (i >> 2) + 2u;
        xwb = (j >> 2) + 2u;
        xa = t4a[qa + min(xwa, la)];
        xb = t4b[qb + min(xwb, lb)];
        st = merge_step();
        if (st != 0) return finish(st);
        ra[slot(ywa)] = ya;
        rb[slot(ywb)] = yb;
        ywa = (i >> 2) + 2u;
        ywb = (j >> 2) + 2u;
        ya = t4a[qa + min(ywa, la)];
        yb = t4b[qb + min(ywb, lb)];
        st = merge_step();
        if (st != 0) return finish(st);
    }
}

// Thread-per-pair verification of the lane's pair (candidate k of request r)
// from its set records: first the head tiles (head_tiles); a pair they leave
// undecided continues from that merge state.  F == 0: in the same lane over
// 16-byte windows of the token array (merge_windows, or with M == kRing
// merge_ring, its loads two steps ahead through the wavefront's window ring);
// with M == kWide only up to here tokens of both sets, longer pairs are queued
// for the deferred kernel.  F > 0: it is appended,
// with its merge state, to the wavefront's list of hard pairs (hcnt entries),
// which groups of F lanes finish (finish_hard), so that no lane walks the token
// array alone while the rest of its wavefront waits.
template <int F, bool C, int M, bool GR>
__device__ __forceinline__ void chunk_thread_pairs(const LaunchArgs& a, const Request& R, int r,
                                                   uint32_t k, bool valid, int2 pr, const LaneRecords& rec,
                                                   bool deferring, uint32_t here, uint32_t* w_defer,
                                                   unsigned long long& dc, int2* w_out, uint32_t& ocnt,
                                                   int2* w_hpr, uint32_t* w_hst, uint32_t& hcnt, uint4* ring) {
    const int lane = lane_id();
    const bool ok = valid && ids_ok(pr, a);
    const uint32_t na = rec.ra0.y, nb = rec.rb0.y;
    const uint32_t L = na + nb;
    const int cls = deferring ? class_of(L, a) : 0;
    const uint32_t alpha = ok ? required_overlap<C>(na, nb, R) : 0u;
    uint32_t i = 0, j = 0, o = 0;
    bool pass = false, act = false;
    auto decide = [&]() {
        pass = ok && o >= alpha;
        act = ok && !pass && o + min(na - i, nb - j) >= alpha;
    };
    const int32_t A[kHeadTokens] = {(int32_t)rec.ra0.z, (int32_t)rec.ra0.w, (int32_t)rec.ra1.x,
                                    (int32_t)rec.ra1.y, (int32_t)rec.ra1.z, (int32_t)rec.ra1.w};
    const int32_t B[kHeadTokens] = {(int32_t)rec.rb0.z, (int32_t)rec.rb0.w, (int32_t)rec.rb1.x,
                                    (int32_t)rec.rb1.y, (int32_t)rec.rb1.z, (int32_t)rec.rb1.w};
    head_tiles(A, B, &i, &j, &o);
    decide();
    // pairs of the deferred classes that the record tokens leave undecided
    const bool defer = act && deferring && cls >= a.defer_from;
    act = act && !defer;
    bool spill = false;
    if constexpr (M == kWide) {
        spill = act && L > here;
        bool cut = false;
        if (act && !spill)
            pass = merge_windows(a.tok, rec.ra0.x, na, a.tok_s, rec.rb0.x, nb, alpha, i, j, o, 0xffffffffu, &cut);
    } else if constexpr (F == 0) {
        const uint32_t budget = deferring ? a.spill_iters : 0xffffffffu;
        if constexpr (M == kRing) {
            if (act)
                pass = merge_ring(a.tok, rec.ra0.x, na, a.tok_s, rec.rb0.x, nb, alpha, i, j, o, budget, &spill,
                                  ring, lane);
        } else {
            if (act) pass = merge_windows(a.tok, rec.ra0.x, na, a.tok_s, rec.rb0.x, nb, alpha, i, j, o, budget, &spill);
        }
    }
    // a spilled merge leaves its state (i, j, o) for the deferred kernel
    if (deferring && spill && a.spill_state != nullptr)
        a.spill_state[a.pair_off[r] + k] = make_uint4(i, j, o, 0u);
    // (after the merges: atomics count with loads, so none sits between the
    // record loads in flight and their use)
    if (ballot(valid && !ok) != 0ull && lane == 0) atomicOr(&a.ctr->err[r], 1u);
    if constexpr (F > 0) {
        const unsigned long long m = ballot(act);
        if (act) {
            const uint32_t pos = hcnt + mbcnt(m);
            w_hpr[pos] = pr;
            w_hst[pos] = i | (j << 8) | (o << 16);  // each <= kHeadTokens
        }
        hcnt += (uint32_t)__popcll(m);
    }
    stage_pass(pass, pr, w_out, ocnt, R.cap == 0);
    if (deferring) {
        defer_pass(a, defer, cls, spill, a.pair_off[r] + k, w_defer, dc);
        note_queued<GR>(a, defer || spill, pr, a.pair_off[r] + k);
    }
}

// Finishes the wavefront's h hard pairs: groups of G lanes resume their
// merges from the saved state with the tile merge.  The loop over the list
// is wave-uniform, so the staging after each step runs with all lanes.
template <int G, bool C>
__device__ __forceinline__ void finish_hard(const LaunchArgs& a, const Request& R, uint32_t h,
                                            const int2* w_hpr, const uint32_t* w_hst, int2* w_out,
                                            uint32_t& ocnt) {
    constexpr uint32_t kGroups = kWave / G;
    const int lane = lane_id();
    const int g = lane % G, gbase = (lane / G) * G;
    const uint32_t grp = (uint32_t)(lane / G);
    wave_sync();
    for (uint32_t e0 = 0; e0 < h; e0 += kGroups) {
        const uint32_t e = e0 + grp;
        bool pass = false;
        int2 pq = make_int2(0, 0);
        if (e < h) {
            pq = w_hpr[e];
            const uint32_t st = w_hst[e];
            const uint2 dr = set_desc(a, pq.x);
            const uint2 ds = set_desc_s(a, pq.y);
            const uint32_t alpha = required_overlap<C>(dr.y, ds.y, R);
            pass = merge_group<G>(a.tok + dr.x, dr.y, a.tok_s + ds.x, ds.y, alpha, g, gbase,
                                  st & 0xffu, (st >> 8) & 0xffu, st >> 16);
        }
        stage_pass(pass && g == 0, pq, w_out, ocnt, R.cap == 0);
    }
    wave_sync();
}

// The walk of a wavefront over its chunks, a lane per pair.  A chunk's pairs
// meet their signatures first, which reject nearly every pair that is not
// similar (of 3.1M candidates of sets of about 12 tokens at 3/5 they leave
// 0.05%, of 620,000 of long sets at 7/10 the wide ones 0.8%, the narrow ones
// 60%).  What they leave is gathered in LDS and verified from the set records
// 64 pairs at a time (chunk_thread_pairs), where no lane idles.  The records
// alone decided so few pairs of a wavefront that every one of them walked
// tokens: two collections 67 -> 40 us, four thresholds 44 -> 34, grouped
// 58 -> 42, 620,000 pairs of long sets 85 -> 36 (their new context's plan
// 198 -> 36), 168M candidates of heavy-tailed sizes 920 -> 768.
//
// What bounds it now is the gather of the signatures.  A 64-lane gather costs
// 2.4 cycles of a compute unit per distinct 128-byte line that the L2 holds and
// 9.4 per line that it does not (measured; a second load from the same line
// 0.7), and the chunks of heavy-tailed sizes meet 31 lines each, of short sets
// 63: hence 16 bytes per set where they do, sets of more than 40 tokens on
// average excepted, whose bitmap of 96 bits would be nearly full.  For the same
// reason chunks and record loads are not split further, and four wavefronts per
// SIMD do as well as six.
//
// Loads never wait for the newest one: candidates are requested three chunks
// ahead and signatures one, into registers that two copies of the step take in
// turn (rotating them by moves waits for the loads), and with the constants of
// the request in scalar registers a chunk of heavy-tailed sizes takes 66 vector
// and 60 scalar instructions instead of 117 and 115.
template <int F, bool D, bool C, int M, bool GR>
__device__ __forceinline__ void walk(const LaunchArgs& a, uint32_t first, uint32_t nw, uint32_t n_chunks,
                                     int2* w_out, uint32_t* w_defer, unsigned long long& dc, int2* w_hpr,
                                     uint32_t* w_hst, int2* w_list, uint32_t* w_list_k, uint32_t* w_marks,
                                     const uint32_t* s_chunk, uint4* w_ring, uint32_t* s_only, uint32_t* s_bad, uint32_t& ocnt, int& r_last) {
    constexpr int U = M == kWide ? kWideUnits : kNarrowUnits;
    // Signatures while they leave at most this many pairs of a chunk on average;
    // otherwise they are tried again on every sixteenth chunk.  (The 18% of the
    // chunks of heavy-tailed sizes that are left many pairs are left 29 of 64:
    // with 24 here the walk took 866 us, with 40 it took 775.)
    constexpr uint32_t kMostLeft = 40;
    // Launches of so few chunks are a chain of memory round trips, to which the
    // narrow signatures add one; their merges run side by side.  With and without
    // them, sets of about 12 tokens: 32,000 pairs 7.5 and 7.0 us, 200,000 11.1 and
    // 10.5; of 30 tokens 32,000 pairs 21.3 and 20.2, 100,000 25.7 and 22.8; of a
    // heavy tail 32,000 13.1 and 12.7, 200,000 20.1 and 19.9; 2,600 pairs of two
    // collections, one call after the other's result, 13.6 and 13.1.
    constexpr uint32_t kFewChunks = 4096;
    // Wide signatures: what they leave is queued, few pairs as a rule, or the long
    // ones at the end of a list whose sets ascend.  A list most of whose pairs are
    // similar is another matter, since a queue takes an atomic per 64 to 128 pairs
    // and the deferred kernel 0.5 ns a pair.  So once a launch has met 2 pairs per
    // chunk, 3%, in lists of kManyPairs and more (counted on kSlots addresses), the
    // lanes merge such a list where it is, except for its pairs of more than a
    // sixteenth of the launch's chunks in tokens: those a lane merges well only
    // while the launch is long against them.  Similar pairs of 130 tokens a set:
    // 20,000 take 48 us queued, and 82 with pairs up to 512 tokens merged here;
    // 600,000 took 371 queued, 217 with up to 256 tokens, 188 with 512, 217 with
    // 1,024; 4,000,000 took 2,140, 1,149, 954 and 843.  600,000 of which half are
    // similar 250 queued, 227 with full lists merged, 156 with those of 32 pairs.
    // Without the count the ends of lists of 620,000 pairs merged here, 70 us
    // instead of 35.  Launches below kManyChunks queue all (their few full lists
    // would only wait for the count: 100,000 pairs 31 us, 35 with it).
    constexpr uint32_t kManyPairs = (uint32_t)kWave / 2u, kManyChunks = 4096;
    const uint32_t sixteenth = n_chunks / 16u;
    bool many = false;
    if (first >= n_chunks) return;
    const int lane = lane_id();
    const bool deferring = D && (a.defer_from < kClasses || spilling(a));
    const bool have = a.sig != nullptr && a.sig_s != nullptr && (M == kWide || n_chunks > kFewChunks);
    const uint4* sig = have ? a.sig : a.heads;
    const uint4* sig_s = have ? a.sig_s : a.heads_s;
    const uint32_t last_r = a.n_sets != 0u ? a.n_sets - 1u : 0u, last_s = a.n_sets_s != 0u ? a.n_sets_s - 1u : 0u;
    const uint32_t share = (n_chunks - 1u - first) / nw + 1u;

    // the request of the chunks whose candidates are requested, and its chunks
    int ri = 0;
    uint32_t bi = 0, ei = a.tile_off[1], ni = a.req[0].n;
    const int2* ci = a.req[0].cand;
    uint32_t ord = 0;  // ordinal of the next chunk to request
    uint32_t vbase = 0, vg = load_chunk_groups<GR>(a, first, nw, n_chunks, 0u, lane, s_chunk);
    // requests the candidates of the next chunk (past the last one: of the last)
    auto issue = [&](CandLoad& c, int& r, uint32_t& kb) {
        const uint32_t q = min(ord++, share - 1u);
        const uint32_t T = first + q * nw;
        while (T >= ei) {
            ++ri;
            bi = ei;
            ei = a.tile_off[ri + 1];
            ni = a.req[ri].n;
            ci = a.req[ri].cand;
        }
        r = ri;
        kb = (T - bi) * (uint32_t)kWave;
        if constexpr (GR) {
            if (q - vbase >= (uint32_t)kWave) {
                vbase = q;
                vg = load_chunk_groups<GR>(a, first, nw, n_chunks, vbase, lane, s_chunk);
            }
            c = issue_cand<GR>(a, a.req[ri], kb, lane, (uint32_t)__builtin_amdgcn_readlane((int)vg, (int)(q - vbase)));
        } else {
            c.p = load_pair(ci, min(kb + (uint32_t)lane, ni - 1u));
        }
    };

    // the request of the chunk being verified
    int rc = 0;
    uint32_t n = 0, num = 0, add = 0, den = 0;
    bool cosine = false;
    uint32_t full = 0;                  // staged pairs that have to leave before more come
    uint32_t left = 0;                  // pairs in the list
    uint32_t left8 = 0;                 // eight times the pairs that recent chunks left
    unsigned long long bad = 0ull;      // lanes that met an id out of range
    auto open_request = [&](int r) {
        rc = r;
        const Request& R = a.req[rc];
        n = R.n;
        num = R.small_num;
        add = R.small_add;
        den = R.small_den;
        if (C && R.rule == kCosine && R.cosine_ratio != 0.0f) {
            cosine = true;
            num = (uint32_t)R.num;
            den = (uint32_t)R.den;
        } else {
            cosine = false;
        }
        full = R.cap == 0 ? 0xffffffffu : wave_stage(M) - kWave;
    };
    // verifies the last m (at most kWave) pairs of the list
    auto finish_list = [&](uint32_t m) {
        wave_sync();
        const bool valid = (uint32_t)lane < m;
        const uint32_t at = left - m + min((uint32_t)lane, m - 1u);
        const int2 pr = w_list[at];
        const uint32_t k = D ? w_list_k[at] : 0u;
        left -= m;
        const Request& R = a.req[rc];
        LaneRecords rec;
        issue_records(a, pr, rec);
        uint32_t hcnt = 0;
        if (M == kWide && m >= kManyPairs && !many && n_chunks >= kManyChunks) {
            uint32_t met = 0;
            if (lane == 0) met = atomicAdd(&a.ctr->slot[blockIdx.x % kSlots].many, m);
            many = (uint32_t)__builtin_amdgcn_readfirstlane((int)met) >= sixteenth;
        }
        chunk_thread_pairs<F, C, M, GR>(a, R, rc, k, valid, pr, rec, deferring, many && m >= kManyPairs ? sixteenth : 0u,
                                        w_defer, dc, w_out, ocnt, w_hpr, w_hst, hcnt, w_ring);
        if constexpr (F > 0)
            if (hcnt != 0u) finish_hard<F, C>(a, R, hcnt, w_hpr, w_hst, w_out, ocnt);
        wave_sync();
    };

    // candidates are requested three chunks ahead, narrow signatures one (wide ones
    // when they are needed: a wavefront has few such chunks, and the 64 registers
    // of two chunks' would leave room for four wavefronts per SIMD instead of five)
    int2 p0;
    int r0, rx, ry;
    uint32_t kb0, kbx, kby;
    CandLoad cx, cy;
    Signatures<kNarrowUnits> qa, qb;
    bool with0 = have;
    {
        CandLoad c0;
        issue(c0, r0, kb0);
        issue(cx, rx, kbx);
        p0 = resolve_cand<GR>(a, a.req[r0], kb0, lane, c0, w_marks);
        if constexpr (M != kWide) issue_signatures<U>(sig, sig_s, with0 ? last_r : 0u, with0 ? last_s : 0u, p0, qa);
        issue(cy, ry, kby);
    }
    // (progress_priority; of wide signatures only in lists that are merged where
    // they are found: 2M candidates of which 0.1% are similar, in shares of 6, 55 us
    // without the steps and 62 with them)
    const bool yields = share >= a.yield_share;
    const uint32_t quarter[3] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)((share + 3u) / 4u)),
                                 (uint32_t)__builtin_amdgcn_readfirstlane((int)((2u * share + 3u) / 4u)),
                                 (uint32_t)__builtin_amdgcn_readfirstlane((int)((3u * share + 3u) / 4u))};
    uint32_t level = 3;
    if (yields && M != kWide) __builtin_amdgcn_s_setprio(3);
    uint32_t done = 0;
    // one chunk: its narrow signatures are in cur, the next chunk's go to nxt; c
    // holds the next chunk's candidates and takes those of the third one
    auto step = [&](Signatures<kNarrowUnits>& cur, Signatures<kNarrowUnits>& nxt, CandLoad& c, int& rn, uint32_t& kbn) {
        if (yields && (M != kWide || many)) progress_priority(done, quarter, level);
        ++done;
        const int2 p1 = resolve_cand<GR>(a, a.req[rn], kbn, lane, c, w_marks);
        const int r1 = rn;
        const uint32_t kb1 = kbn;
        const bool with1 = have && (left8 <= 8u * kMostLeft || (done & 15u) == 0u);
        if constexpr (M != kWide) issue_signatures<U>(sig, sig_s, with1 ? last_r : 0u, with1 ? last_s : 0u, p1, nxt);
        issue(c, rn, kbn);
        const bool valid = kb0 + (uint32_t)lane < n;
        const bool ok = valid && (uint32_t)p0.x < a.n_sets && (uint32_t)p0.y < a.n_sets_s;
        bad |= ballot(valid && !ok);
        bool act = ok;
        if (with0) {
            uint32_t na, nb, most;
            if constexpr (M == kWide) {
                Signatures<U> q;
                issue_signatures<U>(sig, sig_s, last_r, last_s, p0, q);
                na = q.r[0].x, nb = q.s[0].x, most = most_shared<U>(q);
            } else {
                na = cur.r[0].x, nb = cur.s[0].x, most = most_shared<U>(cur);
            }
            if (C && cosine) {
                // (sizes below 2^16, terms below 2^15)
                const uint32_t x = most * den, y = num * num, z = na * nb;
                act = ok && (unsigned long long)x * x >= (unsigned long long)y * z;
            } else if (den != 0u) {
                act = ok && __umul24(most, den) >= __umul24(num, na + nb) + add;
            } else {
                act = ok && most >= (ok ? required_overlap<C>(na, nb, a.req[rc]) : 0u);
            }
        }
        const unsigned long long m = ballot(act);
        const uint32_t more = (uint32_t)__popcll(m);
        if (with0) left8 = left8 - (left8 >> 3) + more;
        if (m != 0ull) {
            if (act) {
                const uint32_t at = left + mbcnt(m);
                w_list[at] = p0;
                if constexpr (D) w_list_k[at] = kb0 + (uint32_t)lane;
            }
            left += more;
        }
        p0 = p1;
        r0 = r1;
        kb0 = kb1;
        with0 = with1;
    };
    // work between chunks: the list is full, another request begins
    auto stop = [&]() {
        return done == share || r0 != rc || left >= (uint32_t)kWave;
    };
    auto between = [&]() {
        const bool close = done == share || r0 != rc;
        while (left >= (close ? 1u : (uint32_t)kWave)) {
            finish_list(min(left, (uint32_t)kWave));
            // (at most kWave staged pairs and entries per queue come at a time)
            if (ocnt > full) {
                wave_flush_out(a, rc, ocnt, w_out, s_only);
                ocnt = 0;
            }
            if (deferring) {
                for (int q = a.defer_from; q < queue_end(a); ++q) {
                    const uint32_t c = dcount(dc, q);
                    if (c > a.defer_cap - kWave) {
                        wave_flush_deferred(a, q, c, w_defer);
                        dc &= ~(0xffull << (8 * q));
                    }
                }
            }
        }
        if (close && bad != 0ull) {
            if (lane == 0) {
                atomicOr(&a.ctr->err[rc], 1u);
                atomicOr(s_bad, 1u << rc);
            }
            bad = 0ull;
        }
        if (close && done != share) {
            if (ocnt != 0u) wave_flush_out(a, rc, ocnt, w_out, s_only);
            ocnt = 0;
            open_request(r0);
        }
    };
    open_request(r0);
    for (;;) {
        step(qa, qb, cx, rx, kbx);
        if (stop()) between();
        if (done == share) break;
        step(qb, qa, cy, ry, kby);
        if (stop()) between();
        if (done == share) break;
    }
    r_last = rc;
}

// ---------------------------------------------------------------------------
// In-order kernel.  Every wavefront takes chunks of kWave consecutive pairs
// of one request, grid-stride over all wavefronts of the grid.  G == 1: a
// lane per pair (walk).  G > 1: 64/G pairs at a time, G lanes each.  D: whether
// the instance can queue pairs for the deferred kernel (an instance without
// that code needs fewer registers).  M: the Mode (G == 1).  GR: a grouped
// launch (every request's candidates read in place from its groups and s ids).
template <int G, int F, bool D, bool C, int M, bool GR>
__global__ __launch_bounds__(kBlock) void k_verify_tiles(LaunchArgs a) {
    touch_args();
    constexpr int GPW = kWave / G;
    constexpr uint32_t kWaves = (uint32_t)(kBlock / kWave);
    // staged output pairs per wavefront: every flush is one atomic on the
    // request's counter, and same-address atomics from all wavefronts are
    // serialised, so flushes carry at least kWStage - kWave pairs
    constexpr uint32_t kWStage = wave_stage(M);
    // the wavefront index is uniform in the wavefront: taken through a scalar
    // register for the chunk walk (which then stays scalar); the LDS
    // addresses use the per-lane copy (vector registers are the cheaper ones)
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t wl = threadIdx.x >> 6;
    const int lane = lane_id();
    const int grp = lane / G, g = lane % G, gbase = grp * G;
    // dynamic LDS, per wavefront: kWStage staged output pairs, then defer_cap
    // entries per queue: the deferred classes q >= defer_from, then the spill
    // queue when merges are cut off (defer_cap >= 2 * kWave)
    extern __shared__ uint4 s_dyn[];
    const bool deferring = D && (a.defer_from < kClasses || spilling(a));
    const uint32_t wave_words =
        (kWStage * 8u +
         (deferring ? (uint32_t)wave_queues(a.defer_from, spilling(a)) * a.defer_cap * 4u : 0u)) / 16u;
    int2* w_out = reinterpret_cast<int2*>(s_dyn + wl * wave_words);
    uint32_t* w_defer = reinterpret_cast<uint32_t*>(w_out + kWStage);
    // hard pairs of the current chunk (thread-per-pair mapping with F > 0)
    __shared__ int2 s_hpr[F > 0 ? kWaves * kWave : 1];
    __shared__ uint32_t s_hst[F > 0 ? kWaves * kWave : 1];
    int2* w_hpr = s_hpr + (F > 0 ? wl * kWave : 0u);
    uint32_t* w_hst = s_hst + (F > 0 ? wl * kWave : 0u);
    // pairs that the signatures leave, and their indices in the request
    __shared__ int2 s_list[G == 1 ? kWaves * 2 * kWave : 1];
    __shared__ uint32_t s_list_k[G == 1 && D ? kWaves * 2 * kWave : 1];
    // group search scratch of grouped launches (resolve_cand)
    __shared__ uint32_t s_marks[GR ? kWaves * kWave : 1];
    uint32_t* w_marks = s_marks + (GR ? wl * kWave : 0u);
    // the chunks' first groups in a small grouped launch
    __shared__ uint32_t s_chunk[GR ? kOwnChunks : 1];
    // the window rings of merge_ring
    __shared__ uint4 s_ring[M == kRing ? kWaves * kRingSlots : 1];
    uint4* w_ring = s_ring + (M == kRing ? wl * kRingSlots : 0u);
    // pairs of the requests without an output buffer, and the wavefronts that
    // have finished
    __shared__ uint32_t s_only[kMaxReq], s_bad, s_finished, s_staged[kWaves], s_staged_req[kWaves];
    __shared__ unsigned long long s_queued[D ? kWaves : 1];  // (dcount)
    int r_last = 0;
    if (threadIdx.x < (unsigned)kMaxReq) s_only[threadIdx.x] = 0u;
    if (threadIdx.x == 0) s_finished = s_bad = 0u;
    if constexpr (GR) {
        if (a.chunk_g == nullptr) {
            // (chunks of a malformed request may get no group: any will do)
            for (uint32_t x = threadIdx.x; x < kOwnChunks; x += (uint32_t)kBlock) s_chunk[x] = 0u;
            __syncthreads();
            for (uint32_t x = threadIdx.x; x < a.group_off[a.n_req]; x += (uint32_t)kBlock)
                group_chunks(a, x, [&](int r, uint32_t t, uint32_t g) { s_chunk[a.tile_off[r] + t] = g; },
                             [&](int r) { atomicOr(&s_bad, 1u << r); });
        }
    }
    __syncthreads();
    uint32_t ocnt = 0;
    unsigned long long dc = 0ull;  // deferred queue fill counts (dcount)
    const uint32_t n_chunks = a.tile_off[a.n_req];
    const uint32_t nw = gridDim.x * kWaves;
    const uint32_t first = blockIdx.x * kWaves + (uint32_t)w;
    if constexpr (G == 1) {
        walk<F, D, C, M, GR>(a, first, nw, n_chunks, w_out, w_defer, dc, w_hpr, w_hst, s_list + wl * 2 * kWave,
                             s_list_k + (D ? wl * 2 * kWave : 0u), w_marks, s_chunk, w_ring, s_only, &s_bad, ocnt, r_last);
    } else {
        int r_cur = 0;
        uint32_t kb_cur = 0;
        if (first < n_chunks) chunk_origin(a, first, &r_cur, &kb_cur);
        const uint32_t share = first < n_chunks ? (n_chunks - 1u - first) / nw + 1u : 1u;
        const uint32_t quarter[3] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)((share + 3u) / 4u)),
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)((2u * share + 3u) / 4u)),
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)((3u * share + 3u) / 4u))};
        uint32_t done = 0, level = 3;
        __builtin_amdgcn_s_setprio(3);
        for (uint32_t T = first; T < n_chunks; T += nw) {
            progress_priority(done++, quarter, level);
            const int r = r_cur;
            const uint32_t kb = kb_cur;
            const uint32_t Tn = T + nw;
            const Request& R = a.req[r];
            if (Tn < n_chunks) chunk_origin(a, Tn, &r_cur, &kb_cur);
            // sub-rounds of 64/G pairs, software-pipelined: while sub-round s
            // is merged, the first tiles of s + 1, the set descriptors of s + 2
            // and the pair of s + 3 are in flight (clamped, unconditional loads
            // keep the issue order fixed)
            // a grouped chunk's pairs are found once, lane k holding pair
            // kb + k, and handed to the groups by permutes
            int2 cp = make_int2(0, 0);
            if constexpr (GR) cp = resolve_cand<GR>(a, R, kb, lane, issue_cand<GR>(a, R, kb, lane, first_group(a, T, s_chunk)), w_marks);
            auto pair_at = [&](int sub) -> int2 {
                const int src = min(sub, G - 1) * GPW + grp;
                if constexpr (GR) return make_int2(bperm(cp.x, src), bperm(cp.y, src));
                const uint32_t k = kb + (uint32_t)src;
                return load_pair(R.cand, k < R.n ? k : R.n - 1);
            };
            auto desc_of = [&](int2 pq, uint2* dr, uint2* ds) {
                const bool ok = ids_ok(pq, a);
                *dr = set_desc(a, ok ? pq.x : 0);
                *ds = set_desc_s(a, ok ? pq.y : 0);
            };
            int2 pq0 = pair_at(0), pq1 = pair_at(1), pq2 = pair_at(2);
            uint2 dr0, ds0, dr1, ds1;
            desc_of(pq0, &dr0, &ds0);
            desc_of(pq1, &dr1, &ds1);
            int32_t wa0 = first_tile_token(a.tok, dr0, g), wb0 = first_tile_token(a.tok_s, ds0, g);
            bool bad = false;
            for (int sub = 0; sub < G; ++sub) {
                const int2 pq3 = pair_at(sub + 3);
                uint2 dr2, ds2;
                desc_of(pq2, &dr2, &ds2);
                const int32_t wa1 = first_tile_token(a.tok, dr1, g);
                const int32_t wb1 = first_tile_token(a.tok_s, ds1, g);
                const uint32_t k = kb + (uint32_t)(sub * GPW + grp);
                bool pass = false, defer = false;
                int cls = 0;
                const int2 pq = pq0;
                if (k < R.n) {
                    if (ids_ok(pq, a)) {
                        const uint32_t L = dr0.y + ds0.y;
                        if (deferring) {
                            cls = class_of(L, a);
                            defer = cls >= a.defer_from;
                        }
                        if (!defer)
                            pass = merge_group_first<G>(a.tok + dr0.x, dr0.y, a.tok_s + ds0.x, ds0.y,
                                                        required_overlap<C>(dr0.y, ds0.y, R), g, gbase,
                                                        wa0, wb0);
                    } else {
                        bad = true;
                    }
                }
                stage_pass(pass && g == 0, pq, w_out, ocnt, R.cap == 0);
                if (deferring) {
                    defer_pass(a, defer && g == 0, cls, false, a.pair_off[r] + k, w_defer, dc);
                    note_queued<GR>(a, defer && g == 0, pq, a.pair_off[r] + k);
                }
                pq0 = pq1;
                pq1 = pq2;
                pq2 = pq3;
                dr0 = dr1;
                ds0 = ds1;
                dr1 = dr2;
                ds1 = ds2;
                wa0 = wa1;
                wb0 = wb1;
            }
            if (ballot(bad) != 0ull && lane == 0) {
                atomicOr(&a.ctr->err[r], 1u);
                atomicOr(&s_bad, 1u << r);
            }
            // at most kWave pairs are staged per chunk: flush when fewer than that
            // fit, or when the next chunk belongs to another request (what is
            // staged after the last chunk goes out with the workgroup's)
            r_last = r;
            const bool other_next = Tn < n_chunks && r_cur != r;
            if (ocnt > 0 && ((R.cap != 0 && ocnt > kWStage - kWave) || other_next)) {
                wave_flush_out(a, r, ocnt, w_out, s_only);
                ocnt = 0;
            }
            if (deferring) {
                // the same bound holds for each queue
                for (int q = a.defer_from; q < queue_end(a); ++q) {
                    const uint32_t c = dcount(dc, q);
                    if (c > a.defer_cap - kWave) {
                        wave_flush_deferred(a, q, c, w_defer);
                        dc &= ~(0xffull << (8 * q));
                    }
                }
            }
        }
    }
    // the workgroup's last wavefront moves what its wavefronts have queued (one
    // atomic per queue) and staged (one for those of the same request, nearly
    // always all), adds the counts and finishes the workgroup.  With an atomic per
    // wavefront, 3.4M pairs that leave something staged in each of 6,144
    // wavefronts spent 50 of 117 us on them, and 636,000 pairs of long sets of
    // which every wavefront queues some 50-70 us, 26-33 with one per workgroup.
    if (ocnt > 0 && a.req[r_last].cap == 0) {
        if (lane == 0) atomicAdd(&s_only[r_last], ocnt);
        ocnt = 0;
    }
    if (lane == 0) {
        s_staged[wl] = ocnt;
        s_staged_req[wl] = (uint32_t)r_last;
        if constexpr (D) s_queued[wl] = dc;
    }
    memory_wait();
    uint32_t fin = 0;
    if (lane == 0) fin = atomicAdd(&s_finished, 1u);
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)fin) != kWaves - 1u) return;
    wave_sync();
    if (deferring) {
        for (int q = a.defer_from; q < queue_end(a); ++q) {
            uint32_t sum = 0;
            for (uint32_t x = 0; x < kWaves; ++x) sum += dcount(s_queued[x], q);
            if (__builtin_amdgcn_readfirstlane((int)sum) == 0) continue;
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&a.ctr->tail[q], sum);
            uint32_t* dst = a.queues + (size_t)q * a.qcap + (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            for (uint32_t x = 0; x < kWaves; ++x) {
                const uint32_t c = dcount(s_queued[x], q);
                const uint32_t* src = reinterpret_cast<const uint32_t*>(s_dyn + x * wave_words) + 2u * kWStage +
                                      (uint32_t)(q - a.defer_from) * a.defer_cap;
                for (uint32_t k = (uint32_t)lane; k < c; k += kWave) dst[k] = src[k];
                dst += c;
            }
        }
    }
    if (quick_end<GR>(a)) {
        // lane r: request r.  The count's address is in the arguments, in host
        // memory: one scalar load, or a vector load on its way with the atomic.
        const bool mine = lane < a.n_req;
        long long* to = nullptr;
        if (a.n_req == 1)
            to = a.req[0].d_count;
        else if (mine)
            to = a.req[lane].d_count;
        uint32_t sum = mine ? s_only[lane] : 0u;
        for (uint32_t q = 0; q < kWaves; ++q) sum += mine && s_staged_req[q] == (uint32_t)lane ? s_staged[q] : 0u;
        const unsigned long long add = (unsigned long long)sum | (1ull << kDoneShift) |
                                       (((s_bad >> (lane & 31)) & 1u) != 0u ? 1ull << kErrShift : 0ull);
        unsigned long long old = 0ull;
        if (mine) old = atomicAdd(&a.ctr->out_count[lane], add);
        uint32_t before[kWaves];  // staged pairs of the same request in the wavefronts before
#pragma unroll
        for (uint32_t q = 0; q < kWaves; ++q) {
            before[q] = 0u;
            for (uint32_t p = 0; p < q; ++p) before[q] += s_staged_req[p] == s_staged_req[q] ? s_staged[p] : 0u;
        }
#pragma unroll
        for (uint32_t q = 0; q < kWaves; ++q) {
            const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_staged[q]);
            if (c == 0u) continue;
            const int rq = __builtin_amdgcn_readfirstlane((int)s_staged_req[q]);
            const unsigned long long base = (((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(old >> 32), rq) << 32 |
                                              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)old, rq)) & kCountMask) + before[q];
            const Request& R = a.req[rq];
            const int2* src = reinterpret_cast<const int2*>(s_dyn + q * wave_words);
            for (uint32_t x = (uint32_t)lane; x < c; x += kWave)
                if (base + x < R.cap) R.out[base + x] = src[x];
        }
        if (mine && ((old >> kDoneShift) & 0xffffull) == gridDim.x - 1u) {
            const unsigned long long all = old + add;
            *to = (all >> kErrShift) != 0ull ? -1ll : (long long)(all & kCountMask);
            a.ctr->out_count[lane] = 0ull;
            a.ctr->err[lane] = 0u;
        }
        return;
    }
    uint32_t left = 0;  // bit q: wavefront q's pairs are still staged
    for (uint32_t q = 0; q < kWaves; ++q) left |= s_staged[q] != 0u ? 1u << q : 0u;
    left = (uint32_t)__builtin_amdgcn_readfirstlane((int)left);
    while (left != 0u) {
        const uint32_t q0 = (uint32_t)__builtin_ctz(left);
        const uint32_t rq = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_staged_req[q0]);
        uint32_t sum = 0;
        for (uint32_t q = q0; q < kWaves; ++q)
            if (((left >> q) & 1u) != 0u && s_staged_req[q] == rq) sum += s_staged[q];
        unsigned long long base = 0ull;
        if (lane == 0) base = atomicAdd(&a.ctr->out_count[rq], (unsigned long long)sum);
        base = lane0_u64(base);
        const Request& R = a.req[rq];
        for (uint32_t q = q0; q < kWaves; ++q) {
            if (((left >> q) & 1u) == 0u || (uint32_t)__builtin_amdgcn_readfirstlane((int)s_staged_req[q]) != rq) continue;
            const uint32_t c = s_staged[q];
            const int2* src = reinterpret_cast<const int2*>(s_dyn + q * wave_words);
            for (uint32_t x = (uint32_t)lane; x < c; x += kWave)
                if (base + x < R.cap) R.out[base + x] = src[x];
            base += c;
            left &= ~(1u << q);
        }
    }
    if (lane < kMaxReq && s_only[lane] != 0u) atomicAdd(&a.ctr->out_count[lane], (unsigned long long)s_only[lane]);
    if (a.two_kernels) return;
    memory_wait();
    finish_workgroup(a);
}

// ---------------------------------------------------------------------------
// Deferred classes, each split statically over all wavefronts of the grid.

// Passing pairs of a wavefront of the deferred kernel, of any requests, in LDS.
constexpr uint32_t kDeferStage = 2 * kWave;
struct DeferStage {
    int2* pr;        // kDeferStage
    uint32_t* req;   // kDeferStage
    uint32_t n;      // wave-uniform
};

// Moves entries [0, n) of a stage to their requests' outputs, with one atomic
// per 64 entries and request.  Called by a whole wavefront.
__device__ void flush_deferred_out(const LaunchArgs& a, const int2* pr, const uint32_t* req, uint32_t n) {
    const int lane = lane_id();
    wave_sync();
    for (uint32_t b = 0; b < n; b += kWave) {
        const uint32_t x = b + (uint32_t)lane;
        const bool have = x < n;
        const int2 p = pr[min(x, n - 1u)];
        const uint32_t r = req[min(x, n - 1u)];
        unsigned long long left = ballot(have);
        while (left != 0ull) {
            const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)r, (int)__builtin_ctzll(left));
            const unsigned long long same = ballot(have && r == r0);
            unsigned long long base = 0ull;
            if (lane == 0) base = atomicAdd(&a.ctr->out_count[r0], (unsigned long long)__popcll(same));
            base = lane0_u64(base) + mbcnt(same);
            if (have && r == r0 && base < a.req[r0].cap) a.req[r0].out[base] = p;
            left &= ~same;
        }
    }
    wave_sync();
}

// Stages the pairs of the lanes with pass set (all lanes of the wavefront
// call it together).
__device__ __forceinline__ void stage_deferred(const LaunchArgs& a, bool pass, int2 pr, int r, DeferStage& s) {
    const unsigned long long m = ballot(pass);
    if (m == 0ull) return;
    if (s.n > kDeferStage - kWave) {
        flush_deferred_out(a, s.pr, s.req, s.n);
        s.n = 0;
    }
    if (pass) {
        s.pr[s.n + mbcnt(m)] = pr;
        s.req[s.n + mbcnt(m)] = (uint32_t)r;
    }
    s.n += (uint32_t)__popcll(m);
}

// A queue whose pairs are merged by a whole wavefront each, with wide tiles (sb:
// kWideTile words), split statically.  The lanes look up 64 of the wavefront's
// pairs side by side, so the chain of queue entry, pair and records is waited
// for once per 64.  (Work stealing costs two accesses to one address per steal,
// about 10 ns each whoever makes them: the pairs above 512 tokens of 620,000
// pairs of long sets took 2.2 ms so, 1.0 ms with a workgroup per pair that
// stole, 83 us without.)
template <bool C, bool GR>
__device__ void drain_wide(const LaunchArgs& a, const Request* reqs, int q, uint32_t cnt, DeferStage& stage,
                           uint32_t* sb) {
    const int lane = lane_id();
    const uint32_t* queue = a.queues + (size_t)q * a.qcap;
    const uint32_t wave = (blockIdx.x * kBlock + threadIdx.x) / kWave;
    const uint32_t waves = gridDim.x * (uint32_t)(kBlock / kWave);
    const bool resume = q == kSpillQ && a.spill_state != nullptr;
    const uint32_t mine = wave < cnt ? (cnt - 1u - wave) / waves + 1u : 0u;
    for (uint32_t b = 0; b < mine; b += kWave) {
        const uint32_t take = min(mine - b, (uint32_t)kWave);
        const uint32_t gi = queue[wave + (b + min((uint32_t)lane, take - 1u)) * waves];
        const int r = request_of_pair(gi, a);
        const int2 pr = queued_pair<GR>(a, reqs, gi, r);
        // (spilled merges resume from their state, as in drain_static)
        const uint4 st = resume ? a.spill_state[gi] : make_uint4(0u, 0u, 0u, 0u);
        const uint2 dr = set_desc(a, pr.x), ds = set_desc_s(a, pr.y);
        const uint32_t alpha = required_overlap<C>(dr.y, ds.y, reqs[r]);
        unsigned long long passed = 0ull;
        for (uint32_t k = 0; k < take; ++k) {
            auto of = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k); };
            if (merge_wide<kWave>(a.tok + of(dr.x), of(dr.y), a.tok_s + of(ds.x), of(ds.y), of(alpha), of(st.x),
                                  of(st.y), of(st.z), lane, 0, sb))
                passed |= 1ull << k;
        }
        stage_deferred(a, ((passed >> lane) & 1ull) != 0ull, pr, r, stage);
    }
}

template <int G, bool C, bool GR>
__device__ void drain_static(const LaunchArgs& a, const Request* reqs, int q, uint32_t cnt, DeferStage& stage,
                             uint32_t* sb) {
    constexpr int GPW = kWave / G;
    const int lane = lane_id();
    const int grp = lane / G, g = lane % G, gbase = grp * G;
    const uint32_t* queue = a.queues + (size_t)q * a.qcap;
    const uint32_t wave = (blockIdx.x * kBlock + threadIdx.x) / kWave;
    const uint32_t stride = (gridDim.x * kBlock) / kWave * GPW;
    const uint32_t t0 = wave * GPW;
    // Item s of the group is queue entry t0 + s * stride + grp.  Software
    // pipeline: while item s is merged, the first tiles of s + 1, the set
    // descriptors of s + 2, the pair of s + 3 and the queue entry of s + 4
    // are in flight (loads clamped to the last entry, so every iteration
    // issues the same loads in the same order).
    auto entry_at = [&](uint32_t s) -> uint32_t {
        const uint32_t k = t0 + s * stride + (uint32_t)grp;
        return queue[min(k, cnt - 1u)];
    };
    // spilled merges resume from the state the in-order kernel left (the
    // merge of the unconsumed suffixes against alpha - o decides the pair the
    // same way: no consumed token matches an unconsumed one)
    const bool resume = q == kSpillQ && a.spill_state != nullptr;
    auto pair_of = [&](uint32_t gi, int* r, uint4* st) -> int2 {
        *r = request_of_pair(gi, a);
        *st = resume ? a.spill_state[gi] : make_uint4(0u, 0u, 0u, 0u);
        return queued_pair<GR>(a, reqs, gi, *r);
    };
    // a set's descriptor without its first c tokens
    auto suffix = [](uint2 d, uint32_t c) { return make_uint2(d.x + c, d.y - c); };
    uint32_t e3;
    int2 p0, p1, p2;
    int r0, r1, r2;
    uint4 st0, st1, st2;
    uint2 dr0, ds0, dr1, ds1;
    int32_t wa0, wb0;
    {
        const uint32_t e0 = entry_at(0), e1 = entry_at(1), e2 = entry_at(2);
        e3 = entry_at(3);
        p0 = pair_of(e0, &r0, &st0);
        p1 = pair_of(e1, &r1, &st1);
        p2 = pair_of(e2, &r2, &st2);
        dr0 = set_desc(a, p0.x);
        ds0 = set_desc_s(a, p0.y);
        dr1 = set_desc(a, p1.x);
        ds1 = set_desc_s(a, p1.y);
        wa0 = first_tile_token(a.tok, suffix(dr0, st0.x), g);
        wb0 = first_tile_token(a.tok_s, suffix(ds0, st0.y), g);
    }
    for (uint32_t t = t0, s = 0; t < cnt; t += stride, ++s) {
        const uint32_t e4 = entry_at(s + 4);
        int r3;
        uint4 st3;
        const int2 p3 = pair_of(e3, &r3, &st3);
        const uint2 dr2 = set_desc(a, p2.x);
        const uint2 ds2 = set_desc_s(a, p2.y);
        const int32_t wa1 = first_tile_token(a.tok, suffix(dr1, st1.x), g);
        const int32_t wb1 = first_tile_token(a.tok_s, suffix(ds1, st1.y), g);
        bool pass = false;
        if (t + (uint32_t)grp < cnt) {
            const uint32_t alpha = required_overlap<C>(dr0.y, ds0.y, reqs[r0]) - st0.z;
            const uint2 ar = suffix(dr0, st0.x), as = suffix(ds0, st0.y);
            const int32_t* A = a.tok + ar.x;
            const int32_t* B = a.tok_s + as.x;
            if constexpr (G == 1) {
                pass = merge_thread(A, ar.y, B, as.y, alpha);
            } else {
                // the tiles in flight first, then wide ones
                pass = alpha == 0u;
                if (!pass && min(ar.y, as.y) >= alpha) {
                    const int ka = (int)min(ar.y, (uint32_t)G), kb = (int)min(as.y, (uint32_t)G);
                    uint32_t i = 0, j = 0, o = 0;
                    group_round<G>(g < ka ? wa0 : 0, g < kb ? wb0 : 0, ka, kb, g, gbase, i, j, o);
                    pass = merge_wide<G>(A, ar.y, B, as.y, alpha, i, j, o, g, gbase, sb + 4 * gbase);
                }
            }
        }
        stage_deferred(a, pass && g == 0, p0, r0, stage);
        e3 = e4;
        p0 = p1;
        r0 = r1;
        st0 = st1;
        p1 = p2;
        r1 = r2;
        st1 = st2;
        p2 = p3;
        r2 = r3;
        st2 = st3;
        dr0 = dr1;
        ds0 = ds1;
        dr1 = dr2;
        ds1 = ds2;
        wa0 = wa1;
        wb0 = wb1;
    }
}

// Lanes per pair of queue q.
__device__ __forceinline__ int lanes_of_queue(const LaunchArgs& a, int q) {
    return q == kSpillQ ? a.spill_lanes : a.lanes[q];
}

// Queues are drained from the spill queue (the longest merges) down to the
// first deferred class.  Four wavefronts per SIMD: left alone the compiler takes
// 164 registers, three wavefronts, and the wide queues are a third slower.
template <bool C, bool GR>
__global__ __launch_bounds__(kBlock, 4) void k_verify_deferred(LaunchArgs a) {
    touch_args();
    constexpr uint32_t kWaves = (uint32_t)(kBlock / kWave);
    static_assert(kWideTile == (uint32_t)kBlock, "the widest mapping is a tile of kBlock tokens");
    __shared__ uint32_t s_tile[kWaves * kWideTile];
    __shared__ int2 s_pr[kWaves * kDeferStage];
    __shared__ uint32_t s_req[kWaves * kDeferStage], s_n[kWaves];
    const uint32_t wl = threadIdx.x / kWave;
    DeferStage stage{s_pr + wl * kDeferStage, s_req + wl * kDeferStage, 0u};
    uint32_t* sb = s_tile + wl * kWideTile;
    // the entries of every queue, looked up side by side
    const uint32_t tails = lane_id() < kQueues ? load_agent(&a.ctr->tail[lane_id()]) : 0u;
    // the requests in LDS: the lanes' pairs are of different requests, and the
    // kernel's arguments lie in host memory, where scalar loads are cached but
    // each vector load goes out
    __shared__ Request s_reqs[kMaxReq];
    if (ballot(tails != 0u) != 0ull) {
        if (threadIdx.x == 0)
            for (int q = 0; q < a.n_req; ++q) s_reqs[q] = a.req[q];
        __syncthreads();
    }
    for (int q = kQueues - 1; q >= 0; --q) {
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)tails, q);
        if (cnt == 0) continue;
        // (of wide signatures: a wavefront each for few pairs, 16 lanes for many;
        // similar pairs of two sets of 130 tokens, a wavefront and 16 lanes: 500 21
        // and 32 us, 4,000 30 and 34, 16,000 34 and 42, 64,000 55 and 54, 120,000 92
        // and 77; the line lies at 16,384 pairs on 256 compute units)
        const int lanes = a.mode != kWide ? lanes_of_queue(a, q) : cnt < gridDim.x * kWaves * 4u ? kBlock : 16;
        switch (lanes) {
            case 1: drain_static<1, C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            case 4: drain_static<4, C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            case 8: drain_static<8, C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            case 16: drain_static<16, C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            case 32: drain_static<32, C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            case 64: drain_static<64, C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            case kBlock: drain_wide<C, GR>(a, s_reqs, q, cnt, stage, sb); break;
            default: break;
        }
    }
    // what the wavefronts have staged, one after the other into the first
    // one's place, leaves with one atomic per request
    if (lane_id() == 0) s_n[wl] = stage.n;
    memory_wait();
    __syncthreads();
    if (wl != 0) return;
    for (uint32_t q = 1; q < kWaves; ++q) {
        const uint32_t c = s_n[q];
        if (c == 0u) continue;
        if (stage.n + c > kDeferStage) {
            flush_deferred_out(a, stage.pr, stage.req, stage.n);
            stage.n = 0;
        }
        for (uint32_t x = (uint32_t)lane_id(); x < c; x += kWave) {
            stage.pr[stage.n + x] = s_pr[q * kDeferStage + x];
            stage.req[stage.n + x] = s_req[q * kDeferStage + x];
        }
        stage.n += c;
        wave_sync();
    }
    if (stage.n > 0u) flush_deferred_out(a, stage.pr, stage.req, stage.n);
    memory_wait();
    finish_workgroup(a);
}

// ---------------------------------------------------------------------------
// Grouped candidates (the interleaved C_O / C form of Sec. 3.3.1): group g is
// {probe id, exclusive end}, and its candidates are the s ids
// sids[end(g-1) .. end(g)) with end(-1) = 0.  The verification kernels read
// them in place (issue_cand / resolve_cand); this pre-pass gives each chunk
// of kWave candidates its first group (group_chunks), in launches too large for
// every workgroup to find them itself.
__global__ void k_group_chunks(LaunchArgs a) {
    const uint32_t total = a.group_off[a.n_req];
    for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < total; x += gridDim.x * blockDim.x)
        group_chunks(a, x, [&](int r, uint32_t t, uint32_t g) { a.req[r].chunk_g[t] = g; }, [](int) {});
}

// Zeroes n 32-bit words (a fill kernel: usable where a memset node is not).
__global__ void k_clear_words(uint32_t* __restrict__ p, uint32_t n) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0u;
}

// Set records from the set lengths (CSR offsets of the caller's layout) and
// the start of each set in the device token array (16-byte aligned).
__global__ void k_build_heads(const int64_t* __restrict__ off, const uint32_t* __restrict__ start,
                              const int32_t* __restrict__ tok, uint4* __restrict__ heads, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t b = start[i];
        const uint32_t len = (uint32_t)(off[i + 1] - off[i]);
        int32_t h[kHeadTokens];
#pragma unroll
        for (int k = 0; k < kHeadTokens; ++k) h[k] = ((uint32_t)k < len) ? tok[b + k] : -1;
        heads[2 * i] = make_uint4(b, len, (uint32_t)h[0], (uint32_t)h[1]);
        heads[2 * i + 1] = make_uint4((uint32_t)h[2], (uint32_t)h[3], (uint32_t)h[4], (uint32_t)h[5]);
    }
}

// Signatures of the sets, narrow and where WIDE wide ones, from the set records:
// 16 lanes per set walk its 16-byte windows and collect its bits in LDS.  (One
// kernel for these and the set records, 16 lanes per set, took 100 us more for
// an upload of 50,000 short sets, this one takes 25.)
template <bool WIDE>
__global__ __launch_bounds__(kBlock) void k_build_signatures(const uint4* __restrict__ heads,
                                                             const int32_t* __restrict__ tok,
                                                             uint4* __restrict__ narrow, uint4* __restrict__ wide,
                                                             int64_t n) {
    constexpr int kLanes = 16, kSets = kBlock / kLanes;
    constexpr uint32_t kNarrowBits = signature_bits(kNarrowUnits), kWideBits = signature_bits(kWideUnits);
    static_assert(4 * kWideUnits <= kLanes, "a lane per word of a signature");
    __shared__ uint32_t s_narrow[kSets][4 * kNarrowUnits], s_wide[WIDE ? kSets : 1][4 * kWideUnits];
    const int w = (int)threadIdx.x / kLanes, g = (int)threadIdx.x % kLanes;
    const uint4* t4 = reinterpret_cast<const uint4*>(tok);
    for (int64_t b = (int64_t)blockIdx.x * kSets; b < n; b += (int64_t)gridDim.x * kSets) {
        const int64_t i = b + w;
        const uint4 h = i < n ? heads[2 * i] : make_uint4(0u, 0u, 0u, 0u);
        const uint32_t len = h.y;
        if (g < 4 * kNarrowUnits) s_narrow[w][g] = g == 0 ? len : 0u;
        if constexpr (WIDE) s_wide[w][g] = g == 0 ? len : 0u;
        wave_sync();
        for (uint32_t x = (uint32_t)g; 4u * x < len; x += kLanes) {
            const uint4 v = t4[(h.x >> 2) + x];
            const uint32_t t[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) {
                if (4u * x + k >= len) break;
                // (multiplicative hashing: Knuth, The Art of Computer Programming, vol. 3, 6.4)
                const uint32_t hash = t[k] * 2654435761u, a = __umulhi(hash, kNarrowBits);
                atomicOr(&s_narrow[w][1u + a / 32u], 1u << (a % 32u));
                if constexpr (WIDE) {
                    const uint32_t c = __umulhi(hash, kWideBits);
                    atomicOr(&s_wide[w][1u + c / 32u], 1u << (c % 32u));
                }
            }
        }
        wave_sync();
        if (i < n && g < kNarrowUnits)
            narrow[i * kNarrowUnits + g] = make_uint4(s_narrow[w][4 * g], s_narrow[w][4 * g + 1], s_narrow[w][4 * g + 2],
                                                      s_narrow[w][4 * g + 3]);
        if constexpr (WIDE) {
            if (i < n && g < kWideUnits)
                wide[i * kWideUnits + g] = make_uint4(s_wide[w][4 * g], s_wide[w][4 * g + 1], s_wide[w][4 * g + 2],
                                                      s_wide[w][4 * g + 3]);
        }
        wave_sync();
    }
}

}  // namespace

bool lanes_supported(int lanes) {
    switch (lanes) {
        case 1: case 4: case 8: case 16: case 32: case 64: case kBlock: return true;
        default: return false;
    }
}

bool inline_supported(int lanes, int hard_lanes) {
    return kernel_verify_tiles(lanes, hard_lanes, kNarrow, false, false, false) != nullptr;
}

template <bool D, bool C, bool GR>
const void* verify_tiles_instance(int lanes, int hard_lanes, int mode) {
    if (mode != kNarrow) {
        if (lanes != 1 || hard_lanes != 0) return nullptr;
        // (wide signatures always queue pairs; no grouped launch has the ring)
        if constexpr (D)
            if (mode == kWide) return (const void*)&k_verify_tiles<1, 0, D, C, kWide, GR>;
        if constexpr (!GR)
            if (mode == kRing) return (const void*)&k_verify_tiles<1, 0, D, C, kRing, GR>;
        return nullptr;
    }
    if (lanes == 1) {
        switch (hard_lanes) {
            case 0: return (const void*)&k_verify_tiles<1, 0, D, C, kNarrow, GR>;
            case 8: return (const void*)&k_verify_tiles<1, 8, D, C, kNarrow, GR>;
            case 16: return (const void*)&k_verify_tiles<1, 16, D, C, kNarrow, GR>;
            default: return nullptr;
        }
    }
    if (hard_lanes != 0) return nullptr;
    switch (lanes) {
        case 4: return (const void*)&k_verify_tiles<4, 0, D, C, kNarrow, GR>;
        case 8: return (const void*)&k_verify_tiles<8, 0, D, C, kNarrow, GR>;
        case 16: return (const void*)&k_verify_tiles<16, 0, D, C, kNarrow, GR>;
        case 32: return (const void*)&k_verify_tiles<32, 0, D, C, kNarrow, GR>;
        case 64: return (const void*)&k_verify_tiles<64, 0, D, C, kNarrow, GR>;
        default: return nullptr;
    }
}

template <bool GR>
const void* verify_tiles_by_flags(int lanes, int hard_lanes, int mode, bool deferring, bool cosine) {
    if (cosine)
        return deferring ? verify_tiles_instance<true, true, GR>(lanes, hard_lanes, mode)
                         : verify_tiles_instance<false, true, GR>(lanes, hard_lanes, mode);
    return deferring ? verify_tiles_instance<true, false, GR>(lanes, hard_lanes, mode)
                     : verify_tiles_instance<false, false, GR>(lanes, hard_lanes, mode);
}

const void* kernel_verify_tiles(int lanes, int hard_lanes, int mode, bool deferring, bool cosine, bool grouped) {
    return grouped ? verify_tiles_by_flags<true>(lanes, hard_lanes, mode, deferring, cosine)
                   : verify_tiles_by_flags<false>(lanes, hard_lanes, mode, deferring, cosine);
}

const void* kernel_verify_deferred(bool cosine, bool grouped) {
    if (grouped)
        return cosine ? (const void*)&k_verify_deferred<true, true> : (const void*)&k_verify_deferred<false, true>;
    return cosine ? (const void*)&k_verify_deferred<true, false> : (const void*)&k_verify_deferred<false, false>;
}

hipError_t launch_group_chunks(const LaunchArgs& a, hipStream_t st) {
    const uint32_t total = a.group_off[a.n_req];
    if (total == 0) return hipSuccess;
    const uint32_t b = std::min<uint32_t>((total + kBlock - 1) / kBlock, 65536u);
    hipLaunchKernelGGL(k_group_chunks, dim3(b), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_build_heads(const int64_t* d_offsets, const uint32_t* d_start, const int32_t* d_tok,
                              uint4* d_heads, int64_t n_sets, hipStream_t st) {
    if (n_sets <= 0) return hipSuccess;
    int64_t blocks = (n_sets + kBlock - 1) / kBlock;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_build_heads, dim3((unsigned)blocks), dim3(kBlock), 0, st, d_offsets, d_start,
                       d_tok, d_heads, n_sets);
    return hipGetLastError();
}

hipError_t launch_build_signatures(const uint4* d_heads, const int32_t* d_tok, uint4* d_narrow, uint4* d_wide,
                                   int64_t n_sets, hipStream_t st) {
    if (n_sets <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<int64_t>((n_sets + 15) / 16, 65536);
    if (d_wide)
        hipLaunchKernelGGL((k_build_signatures<true>), dim3(blocks), dim3(kBlock), 0, st, d_heads, d_tok, d_narrow,
                           d_wide, n_sets);
    else
        hipLaunchKernelGGL((k_build_signatures<false>), dim3(blocks), dim3(kBlock), 0, st, d_heads, d_tok, d_narrow,
                           d_wide, n_sets);
    return hipGetLastError();
}

size_t tiles_lds_bytes(const LaunchArgs& a) {
    // per wavefront: wave_stage staged output pairs, then defer_cap entries
    // per queue (a multiple of 16 bytes)
    const size_t stage = (size_t)wave_stage(a.mode) * sizeof(int2);
    const size_t defer = (size_t)wave_queues(a.defer_from, spilling(a)) * a.defer_cap * 4u;
    return (size_t)(kBlock / kWave) * (stage + defer);
}

hipError_t launch_verify_tiles(const LaunchArgs& a, int grid, hipStream_t st) {
    const void* f = kernel_verify_tiles(a.inline_lanes, a.hard_lanes, a.mode,
                                        a.defer_from < kClasses || spilling(a), a.cosine != 0, a.grouped != 0);
    if (!f) return hipErrorInvalidValue;
    LaunchArgs args = a;
    void* params[] = {&args};
    return hipLaunchKernel(f, dim3((unsigned)grid), dim3(kBlock), params, tiles_lds_bytes(a), st);
}

hipError_t launch_clear_words(uint32_t* d_words, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const size_t b = std::min<size_t>((n + kBlock - 1) / kBlock, 1024);
    hipLaunchKernelGGL(k_clear_words, dim3((unsigned)b), dim3(kBlock), 0, st, d_words, (uint32_t)n);
    return hipGetLastError();
}

hipError_t launch_verify_deferred(const LaunchArgs& a, int grid, hipStream_t st) {
    const void* f = kernel_verify_deferred(a.cosine != 0, a.grouped != 0);
    LaunchArgs args = a;
    void* params[] = {&args};
    return hipLaunchKernel(f, dim3((unsigned)grid), dim3(kBlock), params, 0, st);
}

}  // namespace ssj
