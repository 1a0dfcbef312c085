// Host-side launch helpers of the whole self-join on the GPU (join.hip):
// prefix index, probing and verification without a list of candidates in
// between.  Used by the runtime's ssj_join_device / ssj_join.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssj_device.h"

namespace ssj {

// Counters of one join in flight; every join's last kernel zeroes them again.
struct alignas(64) JoinCtl {
    unsigned long long meets;      // list entries that the probes meet
    unsigned long long all;        // the same without the length bound
    unsigned long long out_count;  // similar pairs appended so far
    unsigned int extra;            // units after the first of their groups
    unsigned int spilled;          // merges cut off by the step budget
    unsigned int done;             // workgroups of k_join_ranges that have finished
    unsigned int pad[7];
};

constexpr uint32_t kUnitMeets = 2048;                        // meetings per work unit
constexpr unsigned long long kMaxMeets = 0x7fffffffull;      // meetings that a join takes
constexpr uint32_t kMaxFirst = 1u << 16;                     // sizes in the table of first entries
constexpr uint32_t kSpillCap = 1u << 18;                     // cut-off merges that are queued

// Whether the totals of a probe pass (meetings, meetings without the length
// bound, over m prefix entries) are within what a join takes.
__host__ __device__ inline bool join_fits(unsigned long long meets, unsigned long long all, uint32_t m) {
    return meets <= kMaxMeets && (unsigned long long)m + all / 64ull < 0x80000000ull;
}

// Work units besides the first of every group of 64 entries that a join of m
// entries can have.
__host__ inline uint32_t join_extra_cap(uint32_t m) {
    const unsigned long long pairs = (unsigned long long)m * m / 2ull;
    return (uint32_t)((pairs < kMaxMeets ? pairs : kMaxMeets) / kUnitMeets) + 1u;
}

struct JoinArgs {
    const uint4* heads;   // set records of the collection
    const int32_t* tok;   // its tokens
    uint32_t n;           // sets
    uint32_t m;           // prefix entries of all sets
    uint32_t key_bits;    // bits of the largest token
    uint32_t sorted;      // != 0: set sizes do not decrease with the id and first holds every size
    unsigned long long num, den;  // t
    Request req;          // overlap rule, output (out, cap, d_count)
    uint32_t* pre;        // n + 1: prefix entries of the sets before
    uint32_t *keys, *keys2, *vals2;  // m each: tokens, sorted tokens, entry numbers in their order
    uint4 *ent, *sent;    // m each: entries in set order, in token order
    uint32_t* lo;         // m: first list entry that the probe meets
    uint32_t* first;      // first entry of the sets of at least this size
    uint2* extra;         // further units: group, first meeting
    uint32_t extra_cap;
    uint4* spill;         // kSpillCap: probe entry, list entry, merge state (i, j)
    uint32_t* spill_o;    // kSpillCap: merge state (o)
    JoinCtl* ctl;
    unsigned long long* h_totals;  // pinned: meets, all
};

// Each call with d_temp null only sets *temp_bytes to the temporary storage
// it needs.
hipError_t join_index(const JoinArgs& a, void* d_temp, size_t* temp_bytes, hipStream_t st);
// Ranges and work units; a.h_totals holds the totals once it has finished.
hipError_t join_ranges(const JoinArgs& a, int n_cu, hipStream_t st);
// Probes, verification, count (nothing but the count -1 where the totals do
// not fit join_fits).
hipError_t join_probe(const JoinArgs& a, int n_cu, hipStream_t st);

}  // namespace ssj
