// Flags fragments over a small join-key domain: no sorts.  The equi-join only
// decides which fact rows count and how often (the number of dim rows with the
// row's key that pass their predicate), so a table over the key domain takes
// its place: one bit per key that a kept dim row has, and the number of
// further rows of a key that repeats.  One pass over the fact columns then
// tests the predicate and the key's bit, reads price, discount and flags of
// the rows that pass in row order, and sums the six groups.
#pragma once
#include "host.hpp"

namespace tqp {

constexpr int FLAGS_GROUPS = 6;
constexpr int FLAGS_PART = FLAGS_GROUPS * 3 + 1;      // sum, count, sum(price) per group; joined rows

// One fragment on the device.  Column pointers start at the fragment's first row.
struct FlagsDirect {
    const int32_t* fk;
    const int32_t* date;
    const int64_t* price;
    const int64_t* disc;
    const int8_t* flagA;
    const int8_t* flagB;
    int64_t n_fact;
    const int32_t* pk;
    const int8_t* seg;
    int64_t n_dim;
    int32_t D;
    int32_t c;
    uint32_t key_mask;
    uint32_t* bits;            // one bit per key value
    uint32_t* extra;           // kept dim rows of a key beyond its first
    uint32_t* repeats;         // nonzero when some key repeats
    int64_t* part;             // [FLAGS_PART][nslot] block sums
    int64_t nslot;
    tqp_flags_out out;
};

// Work items of a batch: rows [r0, r1) of one fragment's fact (or dim) side,
// its block sums in slot `slot`.
struct FlagsItem {
    int32_t frag;
    int32_t slot;
    int64_t r0, r1;
};

constexpr int64_t FLAGS_BATCH_ROWS = 16384;           // fact rows of a batch item
constexpr int64_t FLAGS_BATCH_DIM_ROWS = 1024;        // dim rows of a batch item

// Whether a fragment takes the table (see flags_direct.hip for the rule).
bool flags_direct_ok(const tqp_ctx* ctx, const tqp_flags_fragment& f);
// A batch's tables may take this much more than the row buffers of its sorts:
// what a single fragment's free keys cost at most, sixteen times, or 4 us of
// clearing where the sorts take more launches than that.
constexpr size_t FLAGS_BATCH_SPARE = size_t(16) << 20;
// Whether the fact blocks of a single fragment count its dim rows in LDS.
bool flags_direct_lds(const tqp_flags_fragment& f);
int64_t flags_direct_words(const tqp_flags_fragment& f);      // words of `bits`
void flags_direct_fill(const tqp_flags_fragment& f, const tqp_flags_out& o, FlagsDirect& d);

// One fragment in one launch sequence over the caller's workspace.
tqp_status flags_direct_run(tqp_ctx* ctx, const tqp_flags_fragment& f, const tqp_flags_out& o, void* ws,
                            size_t* ws_bytes, hipStream_t s);
// Many fragments: descriptors and items on the device, the tables cleared by the caller.
tqp_status flags_direct_batch(tqp_ctx* ctx, const FlagsDirect* frags, int nfrag, const FlagsItem* dim_items,
                              int64_t ndim_items, const FlagsItem* fact_items, int64_t nfact_items, hipStream_t s);

}  // namespace tqp
