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
// sets, 52% of a heavy tail's; the two tokens after the meeting, kept with the
// entries, lower the bound by one where they differ (the heavy tail's probe
// kernel 738 -> 427 us).  The others are merged from (i + 1, j + 1) with
// overlap 1, which decides a pair that meets there first.  A pair that passes
// is reported if no common token lies before i and j.
//
// With the set sizes in ascending order (the paper's layout) the sets of one
// size are consecutive and have as many entries each, so everything about an
// entry follows from its number and a table of the sizes, and a probe's list
// starts at the first set that is long enough.  In any other order an entry is
// looked up, and the whole list is walked.
//
// Measured, whole joins on one MI355X, against a counting and a filling pass
// over the lists, a list of candidates and its verification: 100,000 short
// sets at t = 0.6 (3.1M meetings) 1,440 -> 143 us, 50,000 long sets at 0.7
// 3,631 -> 249 us, a heavy tail of 500,000 sets at 0.75 (169M meetings) 13.5
// -> 0.55 ms, 5,000 short sets with the results in host memory 216 -> 110 us.
#include <rocprim/device/device_scan.hpp>
#include <rocprim/iterator/counting_iterator.hpp>
#include <rocprim/iterator/transform_iterator.hpp>

#include "join.h"
#include "merge_device.h"

namespace ssj {
namespace {

constexpr int kSortBlock = 512;                                    // threads of the entry and sort kernels
constexpr uint32_t kSortWaves = (uint32_t)(kSortBlock / kWave);
constexpr uint32_t kSortRows = kSortTile / (uint32_t)kSortBlock;   // items per thread
constexpr uint32_t kEntrySpan = kSortTile / kSortWaves;            // entries per wavefront
constexpr int kClassBlock = 1024;
constexpr int kRangeBlock = 256;
constexpr int kDrainBlock = 1024;
constexpr uint32_t kStage = 256;      // staged output pairs per wavefront
constexpr uint32_t kQueue = 2 * kWave;  // meetings waiting for their merge per wavefront
constexpr uint32_t kMergeBudget = 32;   // window steps before a merge goes to the drain kernel

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

// The sizes of a collection in ascending order: entries before the first set
// of each size, entries per set, and the first entry of the sets that are long
// enough for it (thr); and a coarse index of the sizes by entry number (the
// size of every (1 << lut_shift)-th entry).  One workgroup.
__global__ __launch_bounds__(kClassBlock) void k_join_classes(JoinArgs a) {
    constexpr int kWaves = kClassBlock / kWave;
    __shared__ uint32_t s_sum[kWaves];
    const int lane = lane_id(), w = (int)(threadIdx.x / kWave);
    uint32_t carry = 0;
    for (uint32_t b = 0; b < a.n_classes; b += kClassBlock) {
        const uint32_t c = b + threadIdx.x;
        const bool in = c < a.n_classes;
        const uint4 st = a.classes[in ? c : a.n_classes];
        const uint32_t p = in ? st.y - needed(st.y, a.num, a.den) + 1u : 0u;
        const uint32_t cnt = in ? (a.classes[c + 1u].x - st.x) * p : 0u;
        const uint32_t incl = wave_add_scan(cnt, lane);
        if (lane == kWave - 1) s_sum[w] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (int k = 0; k < kWaves; ++k) {
            before += k < w ? s_sum[k] : 0u;
            carry += s_sum[k];
        }
        if (in) a.cls[c] = make_uint4(before + incl - cnt, st.x, st.y, p);
        __syncthreads();
    }
    if (threadIdx.x == 0) a.cls[a.n_classes] = make_uint4(carry, a.n, 0u, 1u);
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < a.n_classes; c += kClassBlock) {
        const uint4 st = a.classes[c];
        const uint32_t need = needed(st.y, a.num, a.den);
        uint32_t lo = 0, hi = c;  // the first size >= need (need <= its own size)
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2u;
            if (a.cls[mid].z < need)
                lo = mid + 1u;
            else
                hi = mid;
        }
        // division by the entries per set, d: the round-up multiplier of
        // Granlund and Montgomery (PLDI 1994) for 32-bit dividends
        const uint32_t d = a.cls[c].w;
        uint32_t l = 0;
        while (l < 32u && (1ull << l) < d) ++l;
        const unsigned long long magic = (((1ull << l) - d) << 32) / d + 1ull;
        a.cls2[c] = make_uint4(st.z, a.cls[lo].x, (uint32_t)magic, min(l, 1u) | ((max(l, 1u) - 1u) << 8));
    }
    for (uint32_t k = threadIdx.x; k < kLut; k += kClassBlock) {
        const uint32_t e = k << a.lut_shift;
        if (e >= a.m) break;
        uint32_t lo = 0, hi = a.n_classes;  // the last size that begins at or before e
        while (hi - lo > 1u) {
            const uint32_t mid = lo + (hi - lo) / 2u;
            if (a.cls[mid].x <= e)
                lo = mid;
            else
                hi = mid;
        }
        a.lut[k] = lo;
    }
}

// Entry e of a collection with ascending sizes: {set, size, position, index of
// the next token}; *thr receives the first entry that it meets.
__device__ __forceinline__ uint4 entry_of(const JoinArgs& a, uint32_t e, uint32_t* thr) {
    uint32_t c = a.lut[e >> a.lut_shift];
    while (a.cls[c + 1u].x <= e) ++c;
    const uint4 k = a.cls[c];
    const uint4 k2 = a.cls2[c];
    const uint32_t r = e - k.x, t = __umulhi(k2.z, r);
    const uint32_t i = (t + ((r - t) >> (k2.w & 0xffu))) >> (k2.w >> 8), j = r - i * k.w;
    *thr = k2.y;
    return make_uint4(k.y + i, k.z, j, k2.x + i * ((k.z + 3u) & ~3u) + j + 1u);
}

// Adds the workgroup's digit counts to the matrix of counts, one row per
// digit and one column per workgroup.
__device__ __forceinline__ void store_counts(const JoinArgs& a, const uint32_t* hist, uint32_t digits) {
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < digits; d += kSortBlock)
        a.counts[(size_t)d * gridDim.x + blockIdx.x] = hist[d];
}

// Tokens of the entries in set order, and the digit counts of the first sort
// pass.  SORTED: from the table of sizes.  Otherwise each wavefront walks
// kEntrySpan consecutive entries 64 at a time: it finds the set of its first
// entry by a 64-way search of pre, and within 64 entries (of at most 64 sets,
// none of which is without entries) every set marks where it begins and a
// running maximum gives every lane its set; the entries are stored too.  Reads
// and writes are consecutive over the lanes either way (a thread per set wrote
// the 2.0M entries of 50,000 long sets in 173 us; now 12 us).
template <bool SORTED>
__global__ __launch_bounds__(kSortBlock) void k_join_entries(JoinArgs a, uint32_t digits) {
    extern __shared__ uint32_t s_hist[];
    __shared__ uint32_t s_marks[SORTED ? 1 : kSortBlock];
    for (uint32_t d = threadIdx.x; d < digits; d += kSortBlock) s_hist[d] = 0u;
    __syncthreads();
    const int lane = lane_id();
    if constexpr (SORTED) {
#pragma unroll 2
        for (uint32_t k = 0; k < kSortRows; ++k) {
            const uint32_t e = blockIdx.x * kSortTile + k * kSortBlock + threadIdx.x;
            if (e >= a.m) break;
            uint32_t thr;
            const uint32_t key = (uint32_t)a.tok[entry_of(a, e, &thr).w - 1u];
            a.keys[e] = key;
            atomicAdd(&s_hist[key & (digits - 1u)], 1u);
        }
    } else {
        uint32_t* marks = s_marks + (threadIdx.x & ~63u);
        const uint32_t e_begin = blockIdx.x * kSortTile + threadIdx.x / kWave * kEntrySpan;
        const uint32_t e_end = min(a.m, e_begin + kEntrySpan);
        // the set holding e_begin: the largest x with pre[x] <= e_begin
        uint32_t x0 = 0, hi = e_begin < e_end ? a.n : 0u;
        while (hi > x0 + 1u) {
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
                const uint32_t key = (uint32_t)a.tok[start + j];
                a.keys[e] = key;
                a.ent[e] = make_uint4(x0 + o, len, j, start + j + 1u);
                atomicAdd(&s_hist[key & (digits - 1u)], 1u);
            }
            // the set of the next 64's first entry (64 sets from it hold them all)
            x0 += lane_u32(o, kWave - 1);
            if (x0 + 1u < a.n && a.pre[x0 + 1u] <= kb + kWave) ++x0;
        }
    }
    store_counts(a, s_hist, digits);
}

// The sort of the entries by token: least significant digit first, digits of
// up to 10 bits (two passes for up to 1M tokens), each pass a count per digit
// and tile of kSortTile entries, a scan of each digit's row, and a scatter.
// The entries start in set order and every pass keeps the order of equal
// digits, so a list ends up in set order.  Bound by the scattered 8-byte
// writes and by the launches; 2.0M entries of 20 bits: 107 us with rocPRIM's
// radix sort (three passes of 8 bits), 71 us so; 0.54M of 18 bits: 148 us (its
// merge sort) and 35 us.
__global__ __launch_bounds__(kSortBlock) void k_sort_count(JoinArgs a, const uint2* __restrict__ in, uint32_t shift,
                                                           uint32_t digits) {
    extern __shared__ uint32_t s_hist[];
    for (uint32_t d = threadIdx.x; d < digits; d += kSortBlock) s_hist[d] = 0u;
    __syncthreads();
    uint32_t key[kSortRows];
#pragma unroll
    for (uint32_t k = 0; k < kSortRows; ++k) {
        const uint32_t e = blockIdx.x * kSortTile + k * kSortBlock + threadIdx.x;
        key[k] = in[min(e, a.m - 1u)].x;
    }
#pragma unroll
    for (uint32_t k = 0; k < kSortRows; ++k) {
        const uint32_t e = blockIdx.x * kSortTile + k * kSortBlock + threadIdx.x;
        if (e < a.m) atomicAdd(&s_hist[(key[k] >> shift) & (digits - 1u)], 1u);
    }
    store_counts(a, s_hist, digits);
}

// One workgroup per digit: its row of counts becomes the exclusive sums, its
// total goes to totals.
__global__ __launch_bounds__(kBlock) void k_sort_rows(JoinArgs a, uint32_t tiles) {
    constexpr int kWaves = kBlock / kWave;
    __shared__ uint32_t s_sum[kWaves];
    const int lane = lane_id(), w = (int)(threadIdx.x / kWave);
    uint32_t* row = a.counts + (size_t)blockIdx.x * tiles;
    uint32_t carry = 0;
    for (uint32_t b = 0; b < tiles; b += kBlock) {
        const uint32_t k = b + threadIdx.x;
        const uint32_t v = k < tiles ? row[k] : 0u;
        const uint32_t incl = wave_add_scan(v, lane);
        if (lane == kWave - 1) s_sum[w] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (int q = 0; q < kWaves; ++q) {
            before += q < w ? s_sum[q] : 0u;
            carry += s_sum[q];
        }
        if (k < tiles) row[k] = before + incl - v;
        __syncthreads();
    }
    if (threadIdx.x == 0) a.totals[blockIdx.x] = carry;
}

// Moves a tile's entries to their places.  A wavefront ranks its entries 64 at
// a time: the lanes with the same digit find each other by one ballot per
// digit bit, and the wavefront's count of the digit so far (LDS, written by
// the last of them) comes before.  FIRST: the tokens of the entries in set
// order (entry e is item e).
template <bool FIRST>
__global__ __launch_bounds__(kSortBlock) void k_sort_scatter(JoinArgs a, const uint2* __restrict__ in,
                                                             uint2* __restrict__ out, uint32_t shift, uint32_t bits) {
    extern __shared__ uint32_t s_cnt[];  // [kSortWaves][digits]
    __shared__ uint32_t s_sum[kSortWaves];
    const uint32_t digits = 1u << bits;
    const int lane = lane_id();
    const uint32_t w = threadIdx.x / kWave;
    for (uint32_t k = threadIdx.x; k < digits * kSortWaves; k += kSortBlock) s_cnt[k] = 0u;
    uint2 item[kSortRows];
    const uint32_t e0 = blockIdx.x * kSortTile + w * kEntrySpan + (uint32_t)lane;
#pragma unroll
    for (uint32_t k = 0; k < kSortRows; ++k) {
        const uint32_t e = min(e0 + k * kWave, a.m - 1u);
        item[k] = FIRST ? make_uint2(a.keys[e], e) : in[e];
    }
    __syncthreads();
    uint32_t* cnt = s_cnt + w * digits;
    uint32_t rank[kSortRows];
#pragma unroll
    for (uint32_t k = 0; k < kSortRows; ++k) {
        const bool valid = e0 + k * kWave < a.m;
        const uint32_t d = (item[k].x >> shift) & (digits - 1u);
        unsigned long long peers = ballot(valid);
        for (uint32_t b = 0; b < bits; ++b) {
            const bool one = ((d >> b) & 1u) != 0u;
            const unsigned long long m = ballot(one);
            peers &= one ? m : ~m;
        }
        const uint32_t before = cnt[d];
        const uint32_t among = mbcnt(peers), n = (uint32_t)__popcll(peers);
        rank[k] = before + among;
        wave_sync();
        if (valid && among == n - 1u) cnt[d] = before + n;
        wave_sync();
    }
    __syncthreads();
    // the digit's place: smaller digits, earlier tiles, earlier wavefronts
    uint32_t carry = 0;
    for (uint32_t b = 0; b < digits; b += kSortBlock) {
        const uint32_t d = b + threadIdx.x;
        const uint32_t v = d < digits ? a.totals[d] : 0u;
        const uint32_t incl = wave_add_scan(v, lane);
        if (lane == kWave - 1) s_sum[w] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (uint32_t q = 0; q < kSortWaves; ++q) {
            before += q < w ? s_sum[q] : 0u;
            carry += s_sum[q];
        }
        if (d < digits) {
            uint32_t at = before + incl - v + a.counts[(size_t)d * gridDim.x + blockIdx.x];
            for (uint32_t q = 0; q < kSortWaves; ++q) {
                const uint32_t n = s_cnt[q * digits + d];
                s_cnt[q * digits + d] = at;
                at += n;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (uint32_t k = 0; k < kSortRows; ++k) {
        const uint32_t d = (item[k].x >> shift) & (digits - 1u);
        if (e0 + k * kWave < a.m) out[cnt[d] + rank[k]] = item[k];
    }
}

// Smallest list position from which on every entry before q is of q's list
// (token w) and not below entry number thr: doubling steps back from q, then
// bisection.  Within a list the entry numbers ascend.  tile holds the
// list's entries from position b on (most lists begin there).
__device__ __forceinline__ uint32_t list_begin(const uint2* __restrict__ list, const uint2* tile, uint32_t b,
                                               uint32_t q, uint32_t w, uint32_t thr) {
    uint32_t good = q, step = 1, bad = 0;
    bool found = false;  // bad is outside
    auto inside = [&](uint32_t c) {
        const uint2 v = c >= b ? tile[c - b] : list[c];
        return v.x == w && v.y >= thr;
    };
    while (good > 0u) {
        const uint32_t c = good >= step ? good - step : 0u;
        if (inside(c)) {
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
        if (inside(mid))
            good = mid;
        else
            bad = mid;
    }
    return good;
}

// Entries in list order, the range of list entries that each meets, and the
// work units of the probe kernel: a unit is up to kUnitMeets meetings of one
// group of 64 consecutive entries.  The first unit of group g is unit g; groups
// with more meetings append the others to one of kExtraLists lists.  The last
// workgroup to finish stores the number of meetings for the host.  An atomic
// on one address takes about 10 ns whoever issues it, so the lists and the
// counts spread over several (with one address each they took 40 us at 2.0M
// entries and 2,048 workgroups, the rest of the kernel 37 us).
template <bool SORTED>
__global__ __launch_bounds__(kRangeBlock) void k_join_ranges(JoinArgs a, const uint2* __restrict__ list) {
    constexpr int kWaves = kRangeBlock / kWave;
    __shared__ uint2 s_tile[kRangeBlock];
    __shared__ uint32_t s_extra[kWaves];
    __shared__ uint32_t s_base;
    __shared__ unsigned long long s_tot[kWaves];
    const int lane = lane_id(), w = (int)(threadIdx.x / kWave);
    unsigned long long meets = 0ull;
    for (uint32_t b = blockIdx.x * kRangeBlock; b < a.m; b += gridDim.x * kRangeBlock) {
        const uint32_t q = b + threadIdx.x;
        uint32_t cnt = 0;
        const uint2 it = list[min(q, a.m - 1u)];
        s_tile[threadIdx.x] = it;
        __syncthreads();
        if (q < a.m) {
            uint32_t thr = 0;
            const uint4 en = SORTED ? entry_of(a, it.y, &thr) : a.ent[it.y];
            const uint32_t rem = en.y - en.z - 1u;
            // (no token: larger than every token)
            a.sent[q] = make_uint4(en.x, en.y, rem, rem != 0u ? (uint32_t)a.tok[en.w] : 0xffffffffu);
            a.at[q] = en.w;
            const uint32_t lo = list_begin(list, s_tile, b, q, it.x, thr);
            a.lo[q] = lo;
            cnt = q - lo;
        }
        // (cnt < 2^30: the sum of 64 in two halves)
        const unsigned long long T = lane_u32(wave_add_scan(cnt & 0xffffu, lane), kWave - 1) +
                                     ((unsigned long long)lane_u32(wave_add_scan(cnt >> 16, lane), kWave - 1) << 16);
        meets += T;
        const uint32_t more = T > kUnitMeets ? (uint32_t)min((T - 1ull) / kUnitMeets, 0xffffffull) : 0u;
        if (lane == 0) s_extra[w] = more;
        __syncthreads();
        uint32_t before = 0, sum = 0;
        for (int k = 0; k < kWaves; ++k) {
            before += k < w ? s_extra[k] : 0u;
            sum += s_extra[k];
        }
        if (sum > 0u) {  // uniform in the workgroup
            const uint32_t x = blockIdx.x % kExtraLists;
            if (threadIdx.x == 0) s_base = atomicAdd(&a.ctl->slot[x].extra, sum);
            __syncthreads();
            for (uint32_t k = (uint32_t)lane; k < more; k += kWave) {
                const uint32_t at = s_base + before + k;
                if (at < a.extra_cap)
                    a.extra[(size_t)x * a.extra_cap + at] = make_uint2((b / kWave) + (uint32_t)w, (k + 1u) * kUnitMeets);
            }
        }
        __syncthreads();
    }
    if (lane == 0) s_tot[w] = meets;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kWaves; ++k) meets += s_tot[k];
        // one atomic per workgroup, on kSlots addresses, then one per address:
        // the meetings (2^33 stand for more) and the workgroups counted in one
        // word
        const uint32_t slot = blockIdx.x % kSlots;
        const unsigned long long add = (min(meets, 1ull << 33) << 16) + 1ull;
        const unsigned long long sum = atomicAdd(&a.ctl->slot[slot].sum, add) + add;
        const uint32_t of = (gridDim.x - slot + kSlots - 1u) / kSlots, slots = min(gridDim.x, kSlots);
        if ((sum & 0xffffull) == of) {
            const unsigned long long all_add = ((sum >> 16) << 16) + 1ull;
            const unsigned long long all = atomicAdd(&a.ctl->meets, all_add) + all_add;
            if ((all & 0xffffull) == slots) *a.h_meets = all >> 16;
        }
    }
}

// Whether a token is common to A[0, i) and B[0, j), by a merge from their ends
// (an earlier meeting of two similar sets is mostly a few tokens back).
__device__ __forceinline__ bool common_before(const int32_t* __restrict__ A, uint32_t i, const int32_t* __restrict__ B,
                                              uint32_t j) {
    while (i > 0u && j > 0u) {
        const int32_t x = A[i - 1u], y = B[j - 1u];
        if (x == y) return true;
        i -= x > y ? 1u : 0u;
        j -= y > x ? 1u : 0u;
    }
    return false;
}

// Whether the 4-token windows that end before positions i and j (both above 0)
// of the sets at sa and sb share a token before them.  (A token at or after
// position i is not below the token met there, one before j is.)
__device__ __forceinline__ bool common_window(const int32_t* __restrict__ tok, uint32_t sa, uint32_t i, uint32_t sb,
                                              uint32_t j) {
    const uint4* __restrict__ t4 = reinterpret_cast<const uint4*>(tok);
    const uint32_t wa = (i - 1u) >> 2;
    int32_t x[4], y[4];
    unpack_window(t4[(sa >> 2) + wa], x);
    unpack_window(t4[(sb >> 2) + ((j - 1u) >> 2)], y);
    bool hit = false;
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
        bool eq = false;
#pragma unroll
        for (int l = 0; l < 4; ++l) eq |= x[k] == y[l];
        hit |= eq && 4u * wa + k < i;
    }
    return hit;
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

// Probes and merges.  A wavefront takes units of up to kUnitMeets meetings of a
// group of 64 entries and walks them 64 at a time, whatever the lengths of its lists: the
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
    if (!join_fits(load_agent(&a.ctl->meets) >> 16)) return;
    const uint32_t n_groups = (a.m + kWave - 1u) / kWave;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * kWaves + wl));
    // extra units of each list (lane k: list k), and up to its end
    const uint32_t l_extra = lane < (int)kExtraLists ? min(load_agent(&a.ctl->slot[lane].extra), a.extra_cap) : 0u;
    const uint32_t l_ends = wave_add_scan(l_extra, lane);
    const uint32_t n_units = n_groups + lane_u32(l_ends, kWave - 1);
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
        const uint32_t ar = a.at[qq.x], as = a.at[qq.y];
        const uint32_t na = er.y, nb = es.y;
        // merge state after the meeting, and the tokens before it (bi, bj)
        uint32_t i = na - er.z, j = nb - es.z, o = 1u;
        const uint32_t sa = ar - i, sb = as - j;
        const uint32_t bi = i - 1u, bj = j - 1u;
        const uint32_t alpha = required_overlap<false>(na, nb, R);
        bool pass = have && o >= alpha;
        bool spill = false;
        if (have && !pass) {
            // near-copies meet at most of their tokens: where the windows before
            // the meeting share a token, this is not their first (the two loads
            // go out with those of the merge)
            Windows w;
            load_windows(a.tok, sa, na, a.tok, sb, nb, i, j, w);
            bool later = false;
            if (bi > 0u && bj > 0u) later = common_window(a.tok, sa, bi, sb, bj);
            if (!later) pass = merge_loaded(a.tok, sa, na, a.tok, sb, nb, alpha, i, j, o, kMergeBudget, &spill, w);
        }
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
        if (pass && common_before(a.tok + sa, bi, a.tok + sb, bj)) pass = false;
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
            const uint32_t k = u - n_groups;
            const int x = (int)__popcll(ballot(l_ends <= k));  // its list
            const uint2 v = a.extra[(size_t)x * a.extra_cap + (k - (x ? lane_u32(l_ends, x - 1) : 0u))];
            g = v.x;
            begin = v.y;
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
        const uint32_t shift = lo - start;
        uint32_t u_end = 0, u_len = 0, u_rem = 0, u_next = 0, u_shift = 0, u_rank = 0;  // the last step's last probe
        for (uint32_t t0 = begin; t0 < end; t0 += kWave) {
            const uint32_t t = t0 + (uint32_t)lane;
            const bool in = t < end;
            uint32_t r_len, r_rem, r_next, r_rank, s_rank;
            if (u_end >= t0 + kWave) {
                r_len = u_len;
                r_rem = u_rem;
                r_next = u_next;
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
                r_rem = bperm_u32(er.z, own);
                r_next = bperm_u32(er.w, own);
                r_rank = g * kWave + own;
                s_rank = bperm_u32(shift, own) + t;
                const int last = (int)lane_u32(own, kWave - 1);
                u_end = lane_u32(incl, last);
                u_len = lane_u32(er.y, last);
                u_rem = lane_u32(er.z, last);
                u_next = lane_u32(er.w, last);
                u_shift = lane_u32(shift, last);
                u_rank = g * kWave + (uint32_t)last;
            }
            const uint4 es = a.sent[in ? s_rank : rc];
            const uint32_t alpha = required_overlap<false>(r_len, es.y, R);
            // one step of the merge: the lower of the next tokens has no partner
            const uint32_t left = min(r_rem - (r_next < es.w ? 1u : 0u), es.z - (es.w < r_next ? 1u : 0u));
            const bool keep = in && 1u + left >= alpha;
            const unsigned long long mk = ballot(keep);
            if (mk != 0ull) {
                if (keep) queue[qcnt + mbcnt(mk)] = make_uint2(r_rank, s_rank);
                qcnt += (uint32_t)__popcll(mk);
                if (qcnt >= (uint32_t)kWave) merge_queued(kWave);
            }
        }
    }
    if (qcnt > 0u) merge_queued(qcnt);
    // the rest of the workgroup's pairs with one atomic (every wavefront of the
    // grid ends here, and atomics on one address take about 8 ns each)
    __syncthreads();
    uint32_t* ends = reinterpret_cast<uint32_t*>(s_queue);
    if (lane == 0) ends[wl] = ocnt;
    __syncthreads();
    uint32_t before = 0, sum = 0;
    for (uint32_t k = 0; k < (uint32_t)kWaves; ++k) {
        before += k < wl ? ends[k] : 0u;
        sum += ends[k];
    }
    if (sum == 0u) return;
    __shared__ unsigned long long s_base;
    if (threadIdx.x == 0) s_base = atomicAdd(&a.ctl->out_count, (unsigned long long)sum);
    if (R.cap == 0) return;
    __syncthreads();
    for (uint32_t k = (uint32_t)lane; k < ocnt; k += kWave) {
        const unsigned long long to = s_base + before + k;
        if (to < R.cap) R.out[to] = w_out[k];
    }
}

// Merges that the probe kernel cut off, continued by a wavefront per pair; the
// last workgroup to finish publishes the count (-1 where nothing was joined)
// and zeroes the counters.
__global__ __launch_bounds__(kDrainBlock) void k_join_drain(JoinArgs a) {
    __shared__ uint32_t s_tile[kDrainBlock / kWave * kWideTile];
    uint32_t* sb = s_tile + threadIdx.x / kWave * kWideTile;
    const uint32_t cnt = min(load_agent(&a.ctl->spilled), kSpillCap);
    const int g = lane_id();
    const uint32_t waves = gridDim.x * (uint32_t)(kDrainBlock / kWave);
    for (uint32_t k = (blockIdx.x * kDrainBlock + threadIdx.x) / kWave; k < cnt; k += waves) {
        const uint4 st = a.spill[k];
        const uint4 er = a.sent[st.x], es = a.sent[st.y];
        const uint32_t bi = er.y - er.z - 1u, bj = es.y - es.z - 1u;  // tokens before the meeting
        const int32_t* A = a.tok + (a.at[st.x] - bi - 1u);
        const int32_t* B = a.tok + (a.at[st.y] - bj - 1u);
        const uint32_t alpha = required_overlap<false>(er.y, es.y, a.req);
        bool pass = merge_wide<kWave>(A, er.y, B, es.y, alpha, st.z, st.w, a.spill_o[k], g, 0, sb);
        // none of the tokens before may be common
        if (pass && bi > 0u && bj > 0u) pass = !merge_wide<kWave>(A, bi, B, bj, 1u, 0u, 0u, 0u, g, 0, sb);
        if (pass && g == 0) {
            const unsigned long long at = atomicAdd(&a.ctl->out_count, 1ull);
            if (at < a.req.cap) a.req.out[at] = make_int2((int)er.x, (int)es.x);
        }
    }
    memory_wait();
    __syncthreads();
    if (threadIdx.x != 0 || atomicAdd(&a.ctl->drained, 1u) != gridDim.x - 1u) return;
    const bool fits = join_fits(load_agent(&a.ctl->meets) >> 16);
    *a.req.d_count = fits ? (long long)load_agent(&a.ctl->out_count) : -1ll;
    a.ctl->meets = a.ctl->out_count = 0ull;
    a.ctl->spilled = a.ctl->drained = 0u;
    for (uint32_t k = 0; k < kSlots; ++k) {
        a.ctl->slot[k].sum = 0ull;
        a.ctl->slot[k].extra = 0u;
    }
}

// The pieces of every list, counted by the thread at its last entry: entry
// number k of a list has ceil(k / 64), at least one.  Run only where bounds of
// their number do not settle whether the join is refused.
__global__ __launch_bounds__(kBlock) void k_join_pieces(JoinArgs a, const uint2* __restrict__ list) {
    __shared__ unsigned long long s_sum;
    if (threadIdx.x == 0) s_sum = 0ull;
    __syncthreads();
    unsigned long long sum = 0ull;
    for (uint32_t q = blockIdx.x * kBlock + threadIdx.x; q < a.m; q += gridDim.x * kBlock) {
        const uint32_t w = list[q].x;
        if (q + 1u < a.m && list[q + 1u].x == w) continue;
        uint32_t lo = 0, hi = q;  // the list's first entry
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2u;
            if (list[mid].x < w)
                lo = mid + 1u;
            else
                hi = mid;
        }
        const unsigned long long full = (q - lo) / 64u, rest = (q - lo) % 64u;
        sum += 1ull + 32ull * full * (full + 1ull) + rest * (full + 1ull);
    }
    atomicAdd(&s_sum, sum);
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(&a.ctl->pieces, s_sum);
}

}  // namespace

hipError_t join_index(const JoinArgs& a, void* d_temp, size_t* temp_bytes, int n_cu, hipStream_t st) {
    hipError_t e = hipSuccess;
    if (!a.n_classes) {
        auto lengths = rocprim::make_transform_iterator(rocprim::counting_iterator<uint32_t>(0u),
                                                        PrefixLength{a.heads, a.n, a.num, a.den});
        e = rocprim::exclusive_scan(d_temp, *temp_bytes, lengths, a.pre, 0u, (size_t)a.n + 1,
                                    rocprim::plus<uint32_t>(), st);
        if (e != hipSuccess || !d_temp) return e;
    } else {
        if (!d_temp) {
            *temp_bytes = 0;
            return hipSuccess;
        }
        hipLaunchKernelGGL(k_join_classes, dim3(1), dim3(kClassBlock), 0, st, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const uint32_t tiles = join_tiles(a.m);
    const dim3 g(tiles), b(kSortBlock);
    const uint2* in = nullptr;
    uint2* out = a.pairs[0];
    uint32_t shift = 0;
    for (uint32_t pass = 0, left = join_passes(a.key_bits); left > 0u; ++pass, --left) {
        const uint32_t bits = (a.key_bits - shift + left - 1u) / left, digits = 1u << bits;
        if (pass == 0) {
            if (a.n_classes)
                hipLaunchKernelGGL(k_join_entries<true>, g, b, digits * 4u, st, a, digits);
            else
                hipLaunchKernelGGL(k_join_entries<false>, g, b, digits * 4u, st, a, digits);
        } else {
            hipLaunchKernelGGL(k_sort_count, g, b, digits * 4u, st, a, in, shift, digits);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_sort_rows, dim3(digits), dim3(kBlock), 0, st, a, tiles);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const uint32_t lds = digits * kSortWaves * 4u;
        if (pass == 0)
            hipLaunchKernelGGL(k_sort_scatter<true>, g, b, lds, st, a, in, out, shift, bits);
        else
            hipLaunchKernelGGL(k_sort_scatter<false>, g, b, lds, st, a, in, out, shift, bits);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        in = out;
        out = a.pairs[(pass + 1u) & 1u];
        shift += bits;
    }
    const uint32_t rb = (a.m + kRangeBlock - 1u) / kRangeBlock, most = (2048u / kRangeBlock) * (uint32_t)n_cu;
    const dim3 rg(rb < most ? rb : most);
    if (a.n_classes)
        hipLaunchKernelGGL(k_join_ranges<true>, rg, dim3(kRangeBlock), 0, st, a, in);
    else
        hipLaunchKernelGGL(k_join_ranges<false>, rg, dim3(kRangeBlock), 0, st, a, in);
    return hipGetLastError();
}

hipError_t join_probe(const JoinArgs& a, int n_cu, hipStream_t st) {
    // units: the groups and what the larger ones have besides (their number is
    // known on the device only)
    const uint32_t per = kBlock / kWave;
    const unsigned long long units = (unsigned long long)(a.m + kWave - 1u) / kWave + a.extra_cap;
    const unsigned long long b = (units + per - 1u) / per, most = 6ull * (unsigned long long)n_cu;
    hipLaunchKernelGGL(k_join_probe, dim3((unsigned)(b < most ? b : most)), dim3(kBlock), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_join_drain, dim3((unsigned)n_cu), dim3(kDrainBlock), 0, st, a);
    return hipGetLastError();
}

hipError_t join_pieces(const JoinArgs& a, int n_cu, hipStream_t st) {
    const uint2* list = a.pairs[(join_passes(a.key_bits) - 1u) & 1u];
    const uint32_t b = (a.m + kBlock - 1u) / kBlock, most = 8u * (uint32_t)n_cu;
    hipLaunchKernelGGL(k_join_pieces, dim3(b < most ? b : most), dim3(kBlock), 0, st, a, list);
    return hipGetLastError();
}

}  // namespace ssj
