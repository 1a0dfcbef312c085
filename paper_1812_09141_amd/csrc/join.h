// Host-side launch helpers of the whole self-join on the GPU (join.hip):
// prefix index, probing and verification without a list of candidates in
// between.  Used by the runtime's ssj_join_device / ssj_join.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssj_device.h"

namespace ssj {

constexpr uint32_t kExtraLists = 8;
constexpr uint32_t kUnitMeets = 2048;  // meetings per work unit of the probe kernel

// Counters of one join in flight; every join's last kernel zeroes them again.
struct alignas(128) JoinCtl {
    unsigned long long meets;      // list entries that the probes meet, << 16
    unsigned long long out_count;  // similar pairs appended so far
    unsigned int spilled;          // merges cut off by the step budget
    unsigned int drained;          // workgroups of k_join_drain that have finished
    unsigned int pad[2];
    unsigned long long pieces;     // of join_pieces, which the host zeroes
    struct alignas(128) {
        unsigned long long sum;    // meetings << 16, plus the workgroups that counted them
        unsigned int extra;        // units in the extra list of this number
    } slot[kSlots];
};

constexpr unsigned long long kMaxMeets = 0x7fffffffull;      // meetings that a join takes
constexpr uint32_t kSortTile = 4096;                         // entries per workgroup of the sort
constexpr uint32_t kSortBits = 10;                           // most bits per pass
constexpr uint32_t kLut = 1024;                              // coarse index of the set sizes
constexpr uint32_t kSpillCap = 1u << 18;                     // cut-off merges that are queued

// Whether a join with this many meetings is one that the probe kernel takes.
// Host and kernels decide by this alone; m prefix entries have m (m - 1) / 2
// meetings at most.
__host__ __device__ inline bool join_fits(unsigned long long meets) { return meets <= kMaxMeets; }

// A join is refused where its lists, each entry's part below it cut into pieces
// of 64 entries, have 2^31 pieces or more (the work items of the candidates'
// path).  Upper bounds of the pieces: a list of n entries has n + n^2 / 128 at
// most and no more entries than there are sets; and the sets of a list whose
// sizes differ by less than the factor t all meet, so with sizes in at most
// groups such groups it has n^2 / (2 groups) - n / 2 meetings at least.
constexpr unsigned long long kMaxPieces = 1ull << 31;
__host__ inline unsigned long long pieces_of_entries(unsigned long long m, unsigned long long n_sets) {
    return m + m * (m < n_sets ? m : n_sets) / 128ull + 1ull;
}
__host__ inline unsigned long long pieces_of_meetings(unsigned long long meets, uint32_t groups, unsigned long long m) {
    return m + groups * (meets + m / 2ull) / 64ull + 1ull;
}

// Work units besides the first of every group of 64 entries that a join of m
// entries can have.
__host__ inline uint32_t join_extra_cap(uint32_t m) {
    const unsigned long long pairs = (unsigned long long)m * m / 2ull;
    return (uint32_t)((pairs < kMaxMeets ? pairs : kMaxMeets) / kUnitMeets) + 1u;
}

// Workgroups and passes of the sort of m entries by key_bits bits.
__host__ inline uint32_t join_tiles(uint32_t m) { return (m + kSortTile - 1u) / kSortTile; }
__host__ inline uint32_t join_passes(uint32_t key_bits) { return (key_bits + kSortBits - 1u) / kSortBits; }

struct JoinArgs {
    const uint4* heads;   // set records of the collection
    const int32_t* tok;   // its tokens
    uint32_t n;           // sets
    uint32_t m;           // prefix entries of all sets
    uint32_t key_bits;    // bits of the largest token
    // set sizes that do not decrease with the id: the sizes in ascending order,
    // {first set, size, first token's index}, then {n}; else n_classes = 0
    const uint4* classes;
    uint32_t n_classes;
    uint32_t lut_shift;   // (m - 1) >> lut_shift < kLut
    uint4* cls;           // n_classes + 1: {first entry, first set, size, entries per set}
    uint4* cls2;          // n_classes: {first token's index, first entry of the sets met, division by the
                          // entries per set: multiplier and shifts}
    uint32_t* lut;        // kLut
    unsigned long long num, den;  // t
    Request req;          // overlap rule, output (out, cap, d_count)
    uint32_t* pre;        // n + 1: prefix entries of the sets before (n_classes = 0)
    uint4* ent;           // m: entries in set order (n_classes = 0)
    uint32_t* keys;       // m: tokens in set order
    uint2* pairs[2];      // m each: {token, entry} on their way to token order
    uint32_t* counts;     // 2^kSortBits at most x join_tiles(m)
    uint32_t* totals;     // 2^kSortBits
    uint4* sent;          // m: entries in token order: {set, size, tokens after this one, the next token}
    uint32_t* at;         // m: index of that next token
    uint32_t* lo;         // m: first list entry that the probe meets
    uint2* extra;         // kExtraLists lists of extra_cap: further units, {group, first meeting}
    uint32_t extra_cap;
    uint4* spill;         // kSpillCap: probe entry, list entry, merge state (i, j)
    uint32_t* spill_o;    // kSpillCap: merge state (o)
    JoinCtl* ctl;
    unsigned long long* h_meets;   // pinned
};

// Index, ranges and work units; *a.h_meets holds the number of meetings
// once it has finished.  With d_temp null it only sets *temp_bytes to the temporary storage
// it needs.
hipError_t join_index(const JoinArgs& a, void* d_temp, size_t* temp_bytes, int n_cu, hipStream_t st);
// Probes, verification, count (nothing but the count -1 where the meetings do
// not fit join_fits).
hipError_t join_probe(const JoinArgs& a, int n_cu, hipStream_t st);
// Adds the pieces of 64 entries of all lists that join_index has made to
// a.ctl->pieces.
hipError_t join_pieces(const JoinArgs& a, int n_cu, hipStream_t st);

}  // namespace ssj
