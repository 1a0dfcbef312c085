// The whole self-join on the GPU (paper Sec. 2.2 "Filters", Sec. 3.1 AllPairs
// and PPJoin; Definition 1): prefix index, probing and verification in one
// pass over the lists, with no list of candidates in between.
//
// For t = num / den > 0 a set x has p(x) = |x| - ceil(t |x|) + 1 prefix tokens,
// and two similar sets share a token within their prefixes.  An entry is a
// prefix token of a set; entries sorted by (token, set) form one list per
// token, and every unordered pair of entries of a list is a meeting of two
// sets r > s at positions i and j.  A similar pair is found once, at its first
// meeting.  From the first meeting on the overlap is at most
// 1 + min(|r| - i - 1, |s| - j - 1), so a meeting whose bound is below the
// required overlap alpha is dropped on two sizes and two positions alone.
// (That covers the length filter: for |s| < t |r| alpha exceeds |s|.)  This
// leaves 10% of the meetings of short sets at t = 0.6, 12% of those of long
// sets, 52% of a heavy tail's; the others are merged from (i + 1, j + 1) with
// overlap 1, which decides a pair that meets there first.  A pair that passes
// is reported if no common token lies before i and j.
//
// With the set sizes in ascending order (the paper's layout) a probe's list
// starts at the first set that is long enough, found through a table of the
// first entry per size; in any other order the whole list is walked.
//
// Measured, whole joins on one MI355X, against a counting and a filling pass
// over the lists, a list of candidates and its verification: 100,000 short
// sets at t = 0.6 (3.1M meetings) 1,465 -> 272 us, 50,000 long sets at 0.7
// 3,628 -> 319 us, a heavy tail of 500,000 sets at 0.75 (169M meetings) 13.4
// -> 0.93 ms, 5,000 short sets with the results in host memory 220 -> 122 us.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/iterator/counting_iterator.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include "join.h"
#include "merge_device.h"

namespace ssj {
namespace {

constexpr uint32_t kEntrySpan = 512;  // entries per wavefront of k_join_entries
constexpr int kRangeBlock = 1024;
constexpr uint32_t kStage = 256;      // staged output pairs per wavefront
constexpr uint32_t kQueue = 2 * kWave;  // meetings waiting for their merge per wavefront
constexpr uint32_t kMergeBudget = 32;   // window steps before a merge goes to the drain kernel
constexpr uint32_t kBackSteps = 4;      // steps back to an earlier meeting before a merge

__device__ __forceinline__ uint32_t needed(uint32_t len, unsigned long long num, unsigned long long den) {
    return (uint32_t)((num * len + den - 1ull) / den);
}

// Prefix length of set x (0 at x = n, so that the exclusive sum over n + 1
// values ends with the total).
struct PrefixLength {
    const uint4* heads;
    uint32_t n;
    unsigned long long num, den;
    __device__ uint32_t operator()(uint32_t x) const {
        if (x >= n) return 0u;
        const uint32_t len = heads[2 * x].y;
        return len - needed(len, num, den) + 1u;  // t <= 1: at least one
    }
};

// Inclusive sum of v over lanes 0 .. lane of the wavefront.
__device__ __forceinline__ uint32_t wave_add_scan(uint32_t v, int lane) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
    const uint32_t r1 = r0 + (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
    const uint32_t r2 = r1 + (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
    const int row = lane >> 4;
    return v + (row == 0 ? 0u : row == 1 ? r0 : row == 2 ? r1 : r2);
}

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int src) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, src);
}

__device__ __forceinline__ uint32_t bperm_u32(uint32_t v, uint32_t src) { return (uint32_t)bperm((int)v, (int)src); }

// Entries in set order: token and {set, size, position, index of the next
// token} of entry e.  A wavefront writes kEntrySpan consecutive entries, 64
// at a time: it finds the set of its first entry by a 64-way search of pre,
// and within 64 entries (of at most 64 sets, none of which is without
// entries) every set marks where it begins and a running maximum gives every
// lane its set.  Reads and writes are consecutive over the lanes; a thread per
// set wrote the 2.0M entries of 50,000 long sets in 173 us.
__global__ __launch_bounds__(kBlock) void k_join_entries(JoinArgs a) {
    __shared__ uint32_t s_marks[kBlock];
    const int lane = lane_id();
    uint32_t* marks = s_marks + (threadIdx.x & ~63u);
    const uint32_t wave = (blockIdx.x * kBlock + threadIdx.x) / kWave;
    const uint32_t e_begin = wave * kEntrySpan;
    if (e_begin >= a.m) return;
    const uint32_t e_end = min(a.m, e_begin + kEntrySpan);
    // the set holding e_begin: the largest x with pre[x] <= e_begin
    uint32_t x0 = 0, hi = a.n;
    while (hi - x0 > 1u) {
        const uint32_t step = (hi - x0 + 63u) / 64u;
        const uint32_t x = x0 + (uint32_t)lane * step;
        const uint32_t c = (uint32_t)__popcll(ballot(x < hi && a.pre[min(x, a.n)] <= e_begin));
        x0 += (c - 1u) * step;
        hi = min(hi, x0 + step);
    }
    for (uint32_t kb = e_begin; kb < e_end; kb += kWave) {
        const uint32_t xl = min(x0 + (uint32_t)lane, a.n - 1u);
        const bool is_set = x0 + (uint32_t)lane < a.n;
        const uint32_t at = a.pre[xl];
        const uint4 h = a.heads[2 * xl];
        marks[lane] = lane == 0 ? 1u : 0u;
        wave_sync();
        if (is_set && at >= kb && at - kb < (uint32_t)kWave) marks[at - kb] = (uint32_t)lane + 1u;
        wave_sync();
        const uint32_t o = wave_max_scan(marks[lane], lane) - 1u;
        wave_sync();
        const uint32_t e = kb + (uint32_t)lane;
        const uint32_t len = bperm_u32(h.y, o), start = bperm_u32(h.x, o), j = e - bperm_u32(at, o);
        if (e < e_end) {
            a.keys[e] = (uint32_t)a.tok[start + j];
            a.ent[e] = make_uint4(x0 + o, len, j, start + j + 1u);
            if (a.sorted && j == 0u) {
                // the first set of every size above its predecessor's
                const uint32_t x = x0 + o;
                for (uint32_t s = x ? a.heads[2 * (x - 1u)].y + 1u : 0u; s <= len; ++s) a.first[s] = e;
            }
        }
        // the set of the next 64's first entry (64 sets from it hold them all)
        x0 += lane_u32(o, kWave - 1);
        if (x0 + 1u < a.n && a.pre[x0 + 1u] <= kb + kWave) ++x0;
    }
}

// Smallest list position from which on every entry before q is of q's list
// (token w) and not below entry number thr: doubling steps back from q, then
// bisection.  Within a list the entry numbers ascend.
__device__ __forceinline__ uint32_t list_begin(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                               uint32_t q, uint32_t w, uint32_t thr) {
    uint32_t good = q, step = 1, bad = 0;
    bool found = false;  // bad is outside
    while (good > 0u) {
        const uint32_t c = good >= step ? good - step : 0u;
        if (keys[c] == w && vals[c] >= thr) {
            good = c;
            step *= 2u;
        } else {
            bad = c;
            found = true;
            break;
        }
    }
    while (found && good - bad > 1u) {
        const uint32_t mid = bad + (good - bad) / 2u;
        if (keys[mid] == w && vals[mid] >= thr)
            good = mid;
        else
            bad = mid;
    }
    return good;
}

// Waits until every memory operation of the wavefront has completed.
__device__ __forceinline__ void memory_wait() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    return v;
}

// Entries in list order, the range of list entries that each meets, and the
// work units of the probe kernel: a unit is up to kUnitMeets meetings of one
// group of 64 consecutive entries.  The first unit of group g is unit g; the
// few groups with more meetings append the others to extra, reserved with
// one atomic per workgroup and pass.  The last workgroup to finish stores the
// totals for the host (atomics only, each one complete before the next is
// issued, so no fence is needed).
__global__ __launch_bounds__(kRangeBlock) void k_join_ranges(JoinArgs a) {
    constexpr int kWaves = kRangeBlock / kWave;
    __shared__ uint32_t s_extra[kWaves];
    __shared__ uint32_t s_base;
    __shared__ unsigned long long s_tot[2 * kWaves];
    const int lane = lane_id(), w = (int)(threadIdx.x / kWave);
    unsigned long long meets = 0ull, all = 0ull;
    for (uint32_t b = blockIdx.x * kRangeBlock; b < a.m; b += gridDim.x * kRangeBlock) {
        const uint32_t q = b + threadIdx.x;
        unsigned long long cnt = 0ull;
        if (q < a.m) {
            const uint32_t key = a.keys2[q];
            const uint4 en = a.ent[a.vals2[q]];
            a.sent[q] = en;
            const uint32_t thr = a.sorted ? a.first[needed(en.y, a.num, a.den)] : 0u;
            const uint32_t lo = list_begin(a.keys2, a.vals2, q, key, thr);
            a.lo[q] = lo;
            cnt = q - lo;
            if (q + 1u == a.m || a.keys2[q + 1u] != key) {
                const unsigned long long len = q - list_begin(a.keys2, a.vals2, q, key, 0u) + 1ull;
                all += len * (len - 1ull) / 2ull;
            }
        }
        const unsigned long long T = wave_sum_u64(cnt);
        meets += lane == 0 ? T : 0ull;
        const uint32_t more = T > kUnitMeets ? (uint32_t)min((T - 1ull) / kUnitMeets, 0xffffffull) : 0u;
        if (lane == 0) s_extra[w] = more;
        __syncthreads();
        uint32_t before = 0, sum = 0;
        for (int k = 0; k < kWaves; ++k) {
            before += k < w ? s_extra[k] : 0u;
            sum += s_extra[k];
        }
        if (sum > 0u) {  // uniform in the workgroup
            if (threadIdx.x == 0) s_base = atomicAdd(&a.ctl->extra, sum);
            __syncthreads();
            for (uint32_t k = (uint32_t)lane; k < more; k += kWave) {
                const uint32_t slot = s_base + before + k;
                if (slot < a.extra_cap) a.extra[slot] = make_uint2((b / kWave) + (uint32_t)w, (k + 1u) * kUnitMeets);
            }
        }
        __syncthreads();
    }
    all = wave_sum_u64(all);
    if (lane == 0) {
        s_tot[w] = meets;
        s_tot[kWaves + w] = all;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kWaves; ++k) {
            meets += s_tot[k];
            all += s_tot[kWaves + k];
        }
        atomicAdd(&a.ctl->meets, meets);
        atomicAdd(&a.ctl->all, all);
        memory_wait();
        if (atomicAdd(&a.ctl->done, 1u) == gridDim.x - 1u) {
            a.h_totals[0] = atomicAdd(&a.ctl->meets, 0ull);
            a.h_totals[1] = atomicAdd(&a.ctl->all, 0ull);
        }
    }
}

// Steps back from positions (i, j) of two sets through their common tokens:
// whether a token is common to A[0, i) and B[0, j).  After at most limit steps
// it stops with (i, j) where it stopped.
__device__ __forceinline__ bool common_before(const int32_t* __restrict__ A, uint32_t& i,
                                              const int32_t* __restrict__ B, uint32_t& j, uint32_t limit) {
    for (uint32_t s = 0; s < limit && i > 0u && j > 0u; ++s) {
        const int32_t x = A[i - 1u], y = B[j - 1u];
        if (x == y) return true;
        i -= x > y ? 1u : 0u;
        j -= y > x ? 1u : 0u;
    }
    return false;
}

__device__ __forceinline__ uint32_t load_agent(const unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long load_agent(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Moves the wavefront's c staged pairs to the output.
__device__ void flush_pairs(const JoinArgs& a, uint32_t c, const int2* w_out) {
    wave_sync();
    const int lane = lane_id();
    unsigned long long base = 0ull;
    if (lane == 0) base = atomicAdd(&a.ctl->out_count, (unsigned long long)c);
    base = lane0_u64(base);
    if (a.req.cap != 0) {
        for (uint32_t i = (uint32_t)lane; i < c; i += kWave)
            if (base + i < a.req.cap) a.req.out[base + i] = w_out[i];
    }
    wave_sync();
}

// Probes and merges.  A wavefront takes units (k_join_ranges) and walks the
// meetings of a group 64 at a time, whatever the lengths of its lists: the
// meetings of the group's entries are numbered through (a running sum), and
// lane k of a step takes meeting t0 + k.  Where one probe's list covers the
// whole step its values are scalars, else every probe marks where its
// meetings begin and a running maximum gives each lane its probe.  A meeting
// reads 16 consecutive bytes per lane and is dropped or queued (in LDS) on
// sizes and positions; queued meetings are merged 64 at a time, so that the
// lanes of a wavefront that merge are full however few meetings survive.
// Bound by instruction issue: about 40 vector instructions per 64 meetings
// that share a probe, and 250 per 64 merges.
__global__ __launch_bounds__(kBlock) void k_join_probe(JoinArgs a) {
    constexpr int kWaves = kBlock / kWave;
    __shared__ int2 s_out[kWaves * kStage];
    __shared__ uint2 s_queue[kWaves * kQueue];
    __shared__ uint32_t s_marks[kBlock];
    const int lane = lane_id();
    const uint32_t wl = threadIdx.x / kWave;
    int2* w_out = s_out + wl * kStage;
    uint2* queue = s_queue + wl * kQueue;
    uint32_t* marks = s_marks + wl * kWave;
    if (!join_fits(load_agent(&a.ctl->meets), load_agent(&a.ctl->all), a.m)) return;
    const uint32_t n_groups = (a.m + kWave - 1u) / kWave;
    const uint32_t n_units = n_groups + min(load_agent(&a.ctl->extra), a.extra_cap);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * kWaves + wl));
    const Request& R = a.req;
    uint32_t ocnt = 0, qcnt = 0;

    // merges the last n (<= 64) queued meetings
    auto merge_queued = [&](uint32_t n) {
        wave_sync();
        qcnt -= n;
        const bool have = (uint32_t)lane < n;
        const uint2 qq = queue[qcnt + min((uint32_t)lane, n - 1u)];
        wave_sync();
        const uint4 er = a.sent[qq.x], es = a.sent[qq.y];
        const uint32_t na = er.y, nb = es.y;
        const uint32_t sa = er.w - er.z - 1u, sb = es.w - es.z - 1u;
        const uint32_t alpha = required_overlap<false>(na, nb, R);
        uint32_t i = er.z + 1u, j = es.z + 1u, o = 1u;
        uint32_t bi = er.z, bj = es.z;
        bool pass = have && o >= alpha;
        bool act = have && !pass;
        if (have && bi > 0u && bj > 0u && common_before(a.tok + sa, bi, a.tok + sb, bj, kBackSteps)) {
            pass = false;
            act = false;
        }
        bool spill = false;
        if (act) pass = merge_windows(a.tok, sa, na, a.tok, sb, nb, alpha, i, j, o, kMergeBudget, &spill);
        const unsigned long long ms = ballot(spill);
        if (ms != 0ull) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&a.ctl->spilled, (uint32_t)__popcll(ms));
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            const uint32_t slot = base + mbcnt(ms);
            if (spill) {
                if (slot < kSpillCap) {
                    a.spill[slot] = make_uint4(qq.x, qq.y, i, j);
                    a.spill_o[slot] = o;
                } else {  // the queue is full: to the end here
                    bool cut = false;
                    pass = merge_windows(a.tok, sa, na, a.tok, sb, nb, alpha, i, j, o, 0xffffffffu, &cut);
                }
            }
        }
        if (pass && bi > 0u && bj > 0u && common_before(a.tok + sa, bi, a.tok + sb, bj, 0xffffffffu)) pass = false;
        const unsigned long long mp = ballot(pass);
        if (R.cap != 0 && pass) w_out[ocnt + mbcnt(mp)] = make_int2((int)er.x, (int)es.x);
        ocnt += (uint32_t)__popcll(mp);
        if (R.cap != 0 && ocnt > kStage - kWave) {
            flush_pairs(a, ocnt, w_out);
            ocnt = 0;
        }
    };

    for (uint32_t u = wave; u < n_units; u += gridDim.x * kWaves) {
        uint32_t g = u, begin = 0;
        if (u >= n_groups) {
            const uint2 x = a.extra[u - n_groups];
            g = x.x;
            begin = x.y;
        }
        const uint32_t rank = g * kWave + (uint32_t)lane;
        const uint32_t rc = min(rank, a.m - 1u);
        const uint4 er = a.sent[rc];
        const uint32_t lo = a.lo[rc];
        const uint32_t cnt = rank < a.m ? rank - lo : 0u;
        const uint32_t incl = wave_add_scan(cnt, lane);
        const uint32_t start = incl - cnt;  // the probe's first meeting
        const uint32_t T = lane_u32(incl, kWave - 1);
        const uint32_t end = min(T, begin + kUnitMeets);
        const uint32_t rem = er.y - er.z - 1u, shift = lo - start;
        uint32_t u_end = 0, u_len = 0, u_rem = 0, u_shift = 0, u_rank = 0;  // the last step's last probe
        for (uint32_t t0 = begin; t0 < end; t0 += kWave) {
            const uint32_t t = t0 + (uint32_t)lane;
            const bool in = t < end;
            uint32_t r_len, r_rem, r_rank, s_rank;
            if (u_end >= t0 + kWave) {
                r_len = u_len;
                r_rem = u_rem;
                r_rank = u_rank;
                s_rank = u_shift + t;
            } else {
                marks[lane] = 0u;
                wave_sync();
                if (cnt != 0u && start < t0 + kWave && incl > t0) marks[start > t0 ? start - t0 : 0u] = (uint32_t)lane + 1u;
                wave_sync();
                const uint32_t own = wave_max_scan(marks[lane], lane) - 1u;
                wave_sync();
                r_len = bperm_u32(er.y, own);
                r_rem = bperm_u32(rem, own);
                r_rank = g * kWave + own;
                s_rank = bperm_u32(shift, own) + t;
                const int last = (int)lane_u32(own, kWave - 1);
                u_end = lane_u32(incl, last);
                u_len = lane_u32(er.y, last);
                u_rem = lane_u32(rem, last);
                u_shift = lane_u32(shift, last);
                u_rank = g * kWave + (uint32_t)last;
            }
            const uint4 es = a.sent[in ? s_rank : rc];
            const uint32_t alpha = required_overlap<false>(r_len, es.y, R);
            const bool keep = in && 1u + min(r_rem, es.y - es.z - 1u) >= alpha;
            const unsigned long long mk = ballot(keep);
            if (mk != 0ull) {
                if (keep) queue[qcnt + mbcnt(mk)] = make_uint2(r_rank, s_rank);
                qcnt += (uint32_t)__popcll(mk);
                if (qcnt >= (uint32_t)kWave) merge_queued(kWave);
            }
        }
    }
    if (qcnt > 0u) merge_queued(qcnt);
    if (ocnt > 0u) flush_pairs(a, ocnt, w_out);
}

// Merges that the probe kernel cut off, continued by a wavefront per pair.
__global__ __launch_bounds__(kBlock) void k_join_drain(JoinArgs a) {
    constexpr int G = kWave;
    const uint32_t cnt = min(load_agent(&a.ctl->spilled), kSpillCap);
    const int g = lane_id();
    const int gbase = 0;
    for (uint32_t k = (blockIdx.x * kBlock + threadIdx.x) / G; k < cnt; k += gridDim.x * kBlock / G) {
        const uint4 st = a.spill[k];
        const uint4 er = a.sent[st.x], es = a.sent[st.y];
        const int32_t* A = a.tok + (er.w - er.z - 1u);
        const int32_t* B = a.tok + (es.w - es.z - 1u);
        const uint32_t alpha = required_overlap<false>(er.y, es.y, a.req);
        bool pass = merge_group<G>(A, er.y, B, es.y, alpha, g, gbase, st.z, st.w, a.spill_o[k]);
        // (er.z and es.z tokens before the meeting: none may be common)
        if (pass && er.z > 0u && es.z > 0u) pass = !merge_group<G>(A, er.z, B, es.z, 1u, g, gbase);
        if (pass && g == 0) {
            const unsigned long long at = atomicAdd(&a.ctl->out_count, 1ull);
            if (at < a.req.cap) a.req.out[at] = make_int2((int)er.x, (int)es.x);
        }
    }
}

// Publishes the count (-1 where nothing was joined) and zeroes the counters.
__global__ void k_join_finalize(JoinArgs a) {
    if (threadIdx.x == 0) {
        const bool fits = join_fits(a.ctl->meets, a.ctl->all, a.m);
        *a.req.d_count = fits ? (long long)a.ctl->out_count : -1ll;
        a.ctl->meets = a.ctl->all = a.ctl->out_count = 0ull;
        a.ctl->extra = a.ctl->spilled = a.ctl->done = 0u;
    }
}

}  // namespace

hipError_t join_index(const JoinArgs& a, void* d_temp, size_t* temp_bytes, hipStream_t st) {
    auto lengths = rocprim::make_transform_iterator(rocprim::counting_iterator<uint32_t>(0u),
                                                    PrefixLength{a.heads, a.n, a.num, a.den});
    size_t scan_bytes = *temp_bytes, sort_bytes = *temp_bytes;
    auto scan = [&]() {
        return rocprim::exclusive_scan(d_temp, scan_bytes, lengths, a.pre, 0u, (size_t)a.n + 1,
                                       rocprim::plus<uint32_t>(), st);
    };
    // stable, and the entries come in set order: sorted by token alone they
    // are sorted by (token, set)
    auto sort = [&]() {
        return rocprim::radix_sort_pairs(d_temp, sort_bytes, a.keys, a.keys2, rocprim::counting_iterator<uint32_t>(0u),
                                         a.vals2, (size_t)a.m, 0u, a.key_bits, st);
    };
    hipError_t e = scan();
    if (e != hipSuccess) return e;
    if (!d_temp) {
        if ((e = sort()) != hipSuccess) return e;
        *temp_bytes = scan_bytes > sort_bytes ? scan_bytes : sort_bytes;
        return hipSuccess;
    }
    const uint32_t waves = (a.m + kEntrySpan - 1u) / kEntrySpan;
    const uint32_t per = kBlock / kWave;
    hipLaunchKernelGGL(k_join_entries, dim3((waves + per - 1u) / per), dim3(kBlock), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return sort();
}

hipError_t join_ranges(const JoinArgs& a, int n_cu, hipStream_t st) {
    const uint32_t b = (a.m + kRangeBlock - 1u) / kRangeBlock, most = 2u * (uint32_t)n_cu;
    hipLaunchKernelGGL(k_join_ranges, dim3(b < most ? b : most), dim3(kRangeBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t join_probe(const JoinArgs& a, int n_cu, hipStream_t st) {
    // units: the groups and what the larger ones have besides; the extra
    // units' number is known on the device only
    const uint32_t per = kBlock / kWave;
    const unsigned long long units = (unsigned long long)(a.m + kWave - 1u) / kWave + a.extra_cap;
    const unsigned long long b = (units + per - 1u) / per, most = 6ull * (unsigned long long)n_cu;
    hipLaunchKernelGGL(k_join_probe, dim3((unsigned)(b < most ? b : most)), dim3(kBlock), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_join_drain, dim3(8u * (unsigned)n_cu), dim3(kBlock), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_join_finalize, dim3(1), dim3(kWave), 0, st, a);
    return hipGetLastError();
}

}  // namespace ssj
