// Equi-join of a fact side with an int32 column of a dim side, by a table
// over the key domain, grouped by that column: the join and the group-by's
// partition in one pass over the fact rows.
//
//   build   the dim rows (key, group key) partitioned by the top key bits
//           into chunk lists, then one block per slice of at most 2^15 keys collects
//           its rows in LDS and writes the slice of the table whole: per key
//           0 (no dim row), the group key + 1, or, for a key with several dim
//           rows, where their list starts;
//   probe   the fact rows (key, value), partitioned by the top key bits too
//           when the table outgrows an XCD's L2, each read the table once:
//           the table slice of the partitions in work stays in L2.  Matches
//           go straight into the chunk lists of the group partitions; rows
//           whose key has several matches are set aside and expanded by a
//           second kernel, which finds nothing when keys are unique.
//
// The sort-based join this replaces takes two passes over the fact rows, a
// counting pass, an expansion and a pass over its output.
#pragma once
#include <algorithm>

#include "chunks.hpp"
#include "segreduce.hpp"

namespace tqp {

constexpr int TJ_SLICE_LOG2 = 15;                     // most keys per build block: 128 KB of LDS
constexpr int TJ_SLICE = 1 << TJ_SLICE_LOG2;
constexpr uint32_t TJ_LIST = 1u << 31;                // the other bits: start of the key's list
constexpr uint32_t TJ_WIDE = 1u << 30;                // the group key was outside its width (masked)
constexpr int TJ_MAX_GROUP_BITS = 21;
constexpr int TJ_MAX_KEY_BITS = 28;
constexpr int XCDS = 8;
constexpr int TJ_L2_KEY_BITS = 20;                    // a table of 4 MB: probed without a fact partition

struct JoinTable {
    int key_bits = 0;
    int part_bits = 0;                 // of the build's partition
    int slice_bits = 0;                // keys per build block
    uint32_t group_mask = 0;
    uint32_t* slot = nullptr;          // [2^key_bits]
    uint32_t* list = nullptr;          // per key with several rows: their number, then their entries
    uint32_t* list_n = nullptr;        // words of list in use (zero on entry)
    Chunks<uint32_t, uint32_t> rows;
};

// The fact rows whose key has several dim rows: where they lie (the row of
// the source, or the place in the fact partitions' chunks).
struct Spill {
    uint32_t* at = nullptr;
    unsigned long long* n = nullptr;   // zero on entry
};

// Chunks of a probe tile.
template <class V> constexpr int probe_chunks() { return part_tile<V>() / CHUNK; }

template <class V>
struct TableJoin {
    JoinTable t;
    int fact_bits = 0;                 // of the fact partition, 0: none
    int lowb = 0;                      // group-key bits below the group partition
    int dup_blocks = 0;
    Chunks<uint32_t, V> fact;
    Chunks<uint16_t, V> grp;
    Spill spill;
};

// Whether a join of n_fact with n_dim rows over key_bits-bit keys, grouped by
// a column of group_bits bits, takes the table (see tablejoin.hip).
bool table_join_ok(const tqp_ctx* ctx, int64_t n_fact, int64_t n_dim, int key_bits, int group_bits);

// cb: group-key bits (at most TJ_MAX_GROUP_BITS).  spread: how many times the
// inputs' rows the part-filled chunks may hold.  More partitions make better
// work (a build block per partition, more aggregation blocks) and cost
// scratch: callers take the largest spread of TJ_SPREADS whose scratch does
// not exceed that of the sorts.
constexpr int TJ_SPREADS[] = {4, 2, 1};
template <class V>
void table_join_reserve(Arena& a, const tqp_ctx* ctx, TableJoin<V>& j, int64_t n_fact, int64_t n_dim, int key_bits,
                        int cb, int64_t join_cap, bool dim_sorted, int spread) {
    JoinTable& t = j.t;
    t.key_bits = key_bits;
    // 256 slices until a slice outgrows LDS; several slices per partition (each
    // skips the others' rows) where the partitions are fewer
    const int nbd = part_blocks(ctx, n_dim, part_tile<uint32_t>());
    t.part_bits = std::min(key_bits, part_bits_for(spread * n_dim, nbd, PART_MAX_BITS));
    t.slice_bits = std::min(std::max(key_bits - PART_MAX_BITS, 0), TJ_SLICE_LOG2);
    t.slice_bits = std::min(t.slice_bits, key_bits - t.part_bits);
    t.group_mask = key_mask_for(cb);
    t.slot = a.scratch<uint32_t>(int64_t(1) << key_bits);
    t.list = a.scratch<uint32_t>(n_dim + n_dim / 2 + 3);      // 3: a list is read with a word behind it
    t.list_n = a.zero<uint32_t>(1);
    if (!dim_sorted) chunks_reserve(a, t.rows, n_dim, nbd, key_bits, t.part_bits);
    const int nb = part_blocks(ctx, n_fact, part_tile<V>());
    j.fact_bits = key_bits > TJ_L2_KEY_BITS ? part_bits_for(spread * n_fact, nb, PART_MAX_BITS) : 0;
    if (j.fact_bits) chunks_reserve(a, j.fact, n_fact, nb, key_bits, j.fact_bits);
    // the probe over chunk lists has at most a tile per 64 (48) chunks and one
    // more per partition
    int probe_blocks = nb;
    if (j.fact_bits)
        probe_blocks = grid_for(j.fact.nchunk + (int64_t(1) << j.fact_bits) * probe_chunks<V>(), probe_chunks<V>(),
                                (int64_t)ctx->num_cus * PART_BLOCKS_PER_CU);
    if (j.fact_bits) probe_blocks = (probe_blocks + XCDS - 1) / XCDS * XCDS;
    // k_probe_lists: its LDS leaves one block per CU, and its blocks go on with
    // the chunks of the probe's
    j.dup_blocks = std::min(probe_blocks, ctx->num_cus);
    int pb = part_bits_for(spread * join_cap, probe_blocks, PART_MAX_BITS);
    pb = std::min(cb, std::max(pb, cb - BUCKET_LOWB_MAX));
    j.lowb = cb - pb;
    chunks_reserve(a, j.grp, join_cap, probe_blocks, cb, pb);
    j.grp.open = a.scratch<uint32_t>((int64_t)probe_blocks << pb);
    j.spill.at = a.scratch<uint32_t>(n_fact);
    j.spill.n = a.zero<unsigned long long>(1);
}

// ------------------------------------------------------------------ build
// One block per slice.  SORTED: the dim rows are n rows sorted by key, those
// of the slice one range; else the chunk list of the slice's partition, whose
// other slices' rows are skipped.  Bound by latency and by the slices' turns
// (one block of 128 KB LDS per CU, 2^25 keys in 1024 slices): 147 us for 15M
// rows and 128 MB of table, each partition read by its four slices; slices of
// 2^14 keys read every partition twice as often and are slower.
constexpr int TJ_BUILD_BLOCK = 1024;
constexpr int TJ_SAME = 8;             // lanes of a wave with one key from which they are taken together
template <bool SORTED>
__global__ void __launch_bounds__(TJ_BUILD_BLOCK)
k_table_build(JoinTable t, const uint32_t* dkey, const uint32_t* dval, int64_t n) {
    constexpr int W = TJ_BUILD_BLOCK / WAVE, PER = CHUNK / WAVE;
    __shared__ uint32_t s_slot[TJ_SLICE];
    __shared__ int64_t s_range[2];
    __shared__ uint32_t s_many, s_base;
    __shared__ uint32_t s_scan[W];
    const int tid = threadIdx.x, w = tid / WAVE, l = lane_id();
    const uint32_t k0 = blockIdx.x << t.slice_bits, keys = 1u << t.slice_bits;
    const int part = (int)(k0 >> (t.key_bits - t.part_bits));
    if (SORTED) {
        if (w < 2) {
            const int64_t r = wave_bound(dkey, n, k0 + (w ? keys - 1 : 0), w != 0);
            if (l == 0) s_range[w] = r;
        }
    }
    auto clear = [&] {
        for (uint32_t i = tid; i < keys; i += TJ_BUILD_BLOCK) s_slot[i] = 0;
        if (tid == 0) s_many = 0;
        __syncthreads();
    };
    // f(slot, entry, frequent slot) for every dim row of the slice
    auto each = [&](auto f) {
        constexpr int U = 8;                          // loads in flight per thread
        auto enter = [&](const uint32_t (&k)[U], const uint32_t* const (&vp)[U], const bool (&in)[U]) {
            uint32_t v[U];
#pragma unroll
            for (int q = 0; q < U; ++q) v[q] = *vp[q];
            // frequent: the key of the wave's first row, met by several lanes, or ~0
            uint32_t frequent = __builtin_amdgcn_readfirstlane(k[0]);
            if (popc64(ballot(in[0] && k[0] == frequent)) < TJ_SAME) frequent = ~0u;
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (in[q]) f(k[q], ((v[q] & t.group_mask) + 1) | (v[q] & ~t.group_mask ? TJ_WIDE : 0u), frequent);
        };
        uint32_t k[U];
        const uint32_t* vp[U];
        bool in[U];
        if (SORTED) {
            for (int64_t r0 = s_range[0] + w * U * WAVE; r0 < s_range[1]; r0 += W * U * WAVE) {
#pragma unroll
                for (int q = 0; q < U; ++q) {         // clamped index: no branch between the loads
                    const int64_t r = r0 + q * WAVE + l;
                    in[q] = r < s_range[1];
                    const int64_t at = in[q] ? r : s_range[1] - 1;
                    k[q] = dkey[at] - k0;
                    in[q] = in[q] && k[q] < keys;
                    vp[q] = dval + at;
                }
                enter(k, vp, in);
            }
        } else {
            // an even share of the partition's chunks per wave
            constexpr uint32_t C = U / PER;
            const uint32_t nc = t.rows.dcount[part];
            const uint32_t* dir = t.rows.list + t.rows.first[part];
            const uint32_t share = ((nc + W - 1) / W + C - 1) / C * C;
            const uint32_t end = (w + 1) * share < nc ? (w + 1) * share : nc;
            for (uint32_t c0 = w * share; c0 < end; c0 += WAVE) {
                uint32_t id = 0, rows = 0;
                if (c0 + l < end) {
                    id = dir[c0 + l];
                    rows = t.rows.rows[id];
                }
                for (uint32_t g = 0; g < (uint32_t)WAVE && c0 + g < end; g += C) {
#pragma unroll
                    for (int q = 0; q < U; ++q) {     // rows past the end read the chunk's first row
                        const int64_t at = (int64_t)wave_read(id, g + q / PER) * CHUNK;
                        const uint32_t r = (q % PER) * WAVE + l;
                        in[q] = r < wave_read(rows, g + q / PER);
                        k[q] = t.rows.keys[at + (in[q] ? r : 0)] - k0;
                        in[q] = in[q] && k[q] < keys;
                        vp[q] = t.rows.vals + at + (in[q] ? r : 0);
                    }
                    enter(k, vp, in);
                }
            }
        }
    };
    clear();
    each([&](uint32_t k, uint32_t e, uint32_t) {
        if (atomicCAS(&s_slot[k], 0u, e) != 0) s_many = 1;
    });
    __syncthreads();
    if (s_many) {
        // some key has several rows: count the rows of every key, give each
        // such key a list, and enter the rows again.  Lanes with a frequent key
        // are taken together: its slice is one block's work, and its rows would
        // take turns on one LDS word (750k rows with one key: 1944 us one by
        // one, 1161 so).
        __syncthreads();
        clear();
        each([&](uint32_t k, uint32_t, uint32_t frequent) {
            if (frequent == ~0u) {
                atomicAdd(&s_slot[k], 1u);
            } else {
                const uint64_t same = ballot(k == frequent);
                if (k != frequent) atomicAdd(&s_slot[k], 1u);
                else if ((same & lanemask_lt()) == 0) atomicAdd(&s_slot[k], (uint32_t)popc64(same));
            }
        });
        __syncthreads();
        uint32_t mine = 0;
        for (uint32_t i = tid; i < keys; i += TJ_BUILD_BLOCK) mine += s_slot[i] > 1 ? s_slot[i] + 1 : 0;
        uint32_t tot;
        uint32_t off = block_excl_sum<TJ_BUILD_BLOCK>(mine, s_scan, &tot);
        if (tid == 0) s_base = atomicAdd(t.list_n, tot);
        __syncthreads();
        off += s_base;
        // a list is filled from its end: the slot counts down to the place
        // after its number of entries
        for (uint32_t i = tid; i < keys; i += TJ_BUILD_BLOCK) {
            const uint32_t c = s_slot[i];
            if (c > 1) {
                t.list[off] = c;
                off += c + 1;
                s_slot[i] = TJ_LIST | off;
            } else {
                s_slot[i] = 0;
            }
        }
        __syncthreads();
        each([&](uint32_t k, uint32_t e, uint32_t frequent) {
            if (!(s_slot[k] & TJ_LIST)) {
                s_slot[k] = e;
            } else if (frequent == ~0u || k != frequent) {
                t.list[(atomicSub(&s_slot[k], 1u) & ~TJ_LIST) - 1] = e;
            } else {
                const uint64_t same = ballot(true);
                const int lead = __ffsll((unsigned long long)same) - 1;
                uint32_t old = 0;
                if (lane_id() == lead) old = atomicSub(&s_slot[k], (uint32_t)popc64(same));
                old = wave_read(old, lead) & ~TJ_LIST;
                t.list[old - 1 - popc64(same & lanemask_lt())] = e;
            }
        });
        __syncthreads();
        for (uint32_t i = tid; i < keys; i += TJ_BUILD_BLOCK)
            if (s_slot[i] & TJ_LIST) s_slot[i] -= 1;
        __syncthreads();
    }
    for (uint32_t i = tid; i < keys; i += TJ_BUILD_BLOCK) t.slot[k0 + i] = s_slot[i];
}

template <class Src>
tqp_status table_build(tqp_ctx* ctx, hipStream_t s, const JoinTable& t, const Src& src, int64_t n_dim,
                       const char* part_name) {
    tqp_status st = part_launch<uint32_t, uint32_t>(ctx, s, part_name, src, n_dim, t.rows, key_mask_for(t.key_bits),
                                                    "table_list");
    if (st != TQP_OK) return st;
    const int64_t slices = int64_t(1) << (t.key_bits - t.slice_bits);
    TQP_LAUNCH(ctx, s, "table_build",
               k_table_build<false><<<(unsigned)slices, TJ_BUILD_BLOCK, 0, s>>>(t, nullptr, nullptr, 0));
    return TQP_OK;
}
// The dim rows already sorted by key (every key within the width).
inline tqp_status table_build_sorted(tqp_ctx* ctx, hipStream_t s, const JoinTable& t, const uint32_t* dkey,
                                     const uint32_t* dval, int64_t n_dim) {
    const int64_t slices = int64_t(1) << (t.key_bits - t.slice_bits);
    TQP_LAUNCH(ctx, s, "table_build_sorted",
               k_table_build<true><<<(unsigned)slices, TJ_BUILD_BLOCK, 0, s>>>(t, dkey, dval, n_dim));
    return TQP_OK;
}

// ------------------------------------------------------------------ probe
// The table's entry of every row in place of its key (0: no match).
template <class V>
__device__ __forceinline__ void probe_entries(const JoinTable& t, uint32_t (&key)[PartItems<V>::value]) {
#pragma unroll
    for (int j = 0; j < PartItems<V>::value; ++j) {
        const uint32_t e = t.slot[key[j] != PART_NONE ? key[j] : 0u];
        key[j] = key[j] != PART_NONE ? e : 0u;
    }
}
// From the entries to the group keys, or PART_NONE where the row has no match
// or is set aside; place(j) = where item j lies.
template <class V, class Place>
__device__ __forceinline__ void probe_rows(const Spill& sp, uint32_t (&key)[PartItems<V>::value], const Place& place,
                                           bool& wide) {
    constexpr int ITEMS = PartItems<V>::value;
    uint32_t any = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) any |= key[j];
    if (__any((any & (TJ_LIST | TJ_WIDE)) != 0)) {
        // one claim per wave: a device-scope atomic per 64 rows, all on one
        // word, took 6M rows of keys with two dim rows each to 1.6 ms
        uint32_t many = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) many += popc64(ballot((key[j] & TJ_LIST) != 0));
        unsigned long long at = 0;
        if (many && lane_id() == 0) at = atomicAdd(sp.n, (unsigned long long)many);
        at = wave_read(at, 0);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const bool m = (key[j] & TJ_LIST) != 0;
            const uint64_t b = ballot(m);
            if (m) {
                sp.at[at + popc64(b & lanemask_lt())] = place(j);
                key[j] = 0;
            }
            at += popc64(b);
            wide |= (key[j] & TJ_WIDE) != 0;
            key[j] &= ~TJ_WIDE;
        }
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) key[j] -= 1;      // 0, no match: PART_NONE
}

// Short lists are expanded by the probe itself: the tile's rows go into the
// group partitions once per entry, in rounds, instead of through the rows set
// aside (whose keys, slots, lists and values are read again, by a kernel of one
// block per CU).  A round costs a tile's barriers whatever it holds, so that
// lists of up to TJ_SHORT entries take part where a sixteenth of the tile's rows
// have the longest of them.  Every key on two dim rows, 40M x 10M rows: 1681
// us, 6M x 1.5M 327, on three 405, on four 424; set aside 2487, 498, 512 and 526, by
// the sorts 1733, 459, 533 and 627.
constexpr uint32_t TJ_SHORT = 4;
constexpr int TJ_SHORT_SHARE = 16;

// The longest lists to expand in place, 0 (none) or 2 to TJ_SHORT, by each
// wave's first 64 rows.  Called by the whole block.
template <class V>
__device__ __forceinline__ uint32_t short_lists(const JoinTable& t, const uint32_t (&key)[PartItems<V>::value],
                                                uint32_t (&s_len)[PART_BLOCK / WAVE]) {
    const bool m = (key[0] & TJ_LIST) != 0;
    const uint32_t len = t.list[m ? key[0] & ~TJ_LIST : 0u];
    uint32_t n = 0;                    // rows with lists of 2, 3, 4 entries, 10 bits each
#pragma unroll
    for (uint32_t q = 0; q <= TJ_SHORT - 2; ++q) n |= (uint32_t)popc64(ballot(m && len == q + 2)) << (10 * q);
    if (lane_id() == 0) s_len[threadIdx.x / WAVE] = n;
    __syncthreads();
    n = 0;
#pragma unroll
    for (int w = 0; w < PART_BLOCK / WAVE; ++w) n += s_len[w];
    uint32_t longest = 0;
#pragma unroll
    for (uint32_t q = 0; q <= TJ_SHORT - 2; ++q)
        if ((n >> (10 * q) & 1023) >= PART_BLOCK / TJ_SHORT_SHARE) longest = q + 2;
    return __builtin_amdgcn_readfirstlane(longest);
}
// Of the tile's lists of at most `longest` entries, entries r and r + 1 (0 past
// their end), read together: a second read of lists beyond the caches costs
// more than the registers.  In round 0 the other rows' entries too, in out.
template <class V>
__device__ __forceinline__ void round_entries(const JoinTable& t, const uint32_t (&key)[PartItems<V>::value],
                                              uint32_t r, uint32_t longest, uint32_t (&out)[PartItems<V>::value],
                                              uint32_t (&next)[PartItems<V>::value]) {
    constexpr int ITEMS = PartItems<V>::value, FLIGHT = 4;     // read together
#pragma unroll
    for (int j0 = 0; j0 < ITEMS; j0 += FLIGHT) {
        struct List { uint32_t n, e[2]; } x[FLIGHT];           // one read in round 0
        uint32_t k[FLIGHT];
#pragma unroll
        for (int j = 0; j < FLIGHT; ++j) {
            k[j] = key[j0 + j];
            asm volatile("" : "+v"(k[j]));             // opaque: no address is kept from round to round
            const uint32_t at = k[j] & TJ_LIST ? k[j] & ~TJ_LIST : 0u;
            __builtin_memcpy(&x[j], t.list + at, sizeof(List));
            if (r) __builtin_memcpy(x[j].e, t.list + (x[j].n > r ? at + 1 + r : at), sizeof x[j].e);
        }
#pragma unroll
        for (int j = 0; j < FLIGHT; ++j) {
            const bool mine = (k[j] & TJ_LIST) && x[j].n <= longest;
            out[j0 + j] = mine ? (r < x[j].n ? x[j].e[0] : 0u) : r ? 0u : k[j];
            next[j0 + j] = mine && r + 1 < x[j].n ? x[j].e[1] : 0u;
        }
        asm volatile("" ::: "memory");
    }
}

// What a probe kernel is for: any table (its lists set aside); or, from 2^22
// rows on, one kernel for a table of unique keys and one for a table with lists,
// of which one returns at once.  In one kernel the registers of the second cost
// the first 2 to 14%.  A launch for nothing costs 3 to 5 us, 3 to 5% of what 3M
// rows take, where the lists set aside cost less than the sorts (3M x 750k rows
// of keys with two dim rows each: 296 and 324 us; 4.1M 359 and 368; 4.3M 302 by
// the kernel for lists, 382 set aside).
enum : int { PROBE_ANY = 0, PROBE_UNIQUE = 1, PROBE_LISTS = 2 };
constexpr int64_t TJ_SHORT_ROWS = int64_t(1) << 22;

// The tile's entries into the group partitions.
template <int MODE, class V, class Place>
__device__ __forceinline__ void probe_tile(const JoinTable& t, const Spill& sp, const Chunks<uint16_t, V>& out,
                                           int parts, uint32_t (&key)[PartItems<V>::value],
                                           const V (&val)[PartItems<V>::value], const Place& place, bool& wide,
                                           PartSmem<V>& sm, uint32_t (&s_len)[PART_BLOCK / WAVE]) {
    probe_entries<V>(t, key);
    if constexpr (MODE == PROBE_LISTS) {
        const uint32_t longest = short_lists<V>(t, key, s_len);
        uint32_t r = 0;
        uint32_t entry[PartItems<V>::value], next[PartItems<V>::value];
        do {
            if (r & 1) {
#pragma unroll
                for (int j = 0; j < PartItems<V>::value; ++j) entry[j] = next[j];
            } else if (longest) {
                round_entries<V>(t, key, r, longest, entry, next);
            } else {
#pragma unroll
                for (int j = 0; j < PartItems<V>::value; ++j) entry[j] = key[j];
            }
            probe_rows<V>(sp, entry, place, wide);
            part_tile_rows<uint16_t, V, PART_BLOCK>(out, parts, entry, val, sm);
        } while (++r < longest);
    } else {
        probe_rows<V>(sp, key, place, wide);
        part_tile_rows<uint16_t, V, PART_BLOCK>(out, parts, key, val, sm);
    }
}

// The probe over a fact source's rows (a table that fits L2).
template <class V, class Src, int MODE>
__global__ void __launch_bounds__(PART_BLOCK, PART_WAVES)
k_probe_cols(Src src, JoinTable t, Spill sp, Chunks<uint16_t, V> out, int parts, uint32_t* flags) {
    constexpr int ITEMS = PartItems<V>::value, TILE = PART_BLOCK * ITEMS;
    __shared__ PartSmem<V> sm;
    __shared__ uint32_t s_len[PART_BLOCK / WAVE];
    if (MODE != PROBE_ANY && (*t.list_n != 0) != (MODE == PROBE_LISTS)) return;
    const int w = wave_index(), l = lane_id();
    part_init<uint16_t, V, PART_BLOCK>(sm);
    const int64_t n = src.size();
    const int64_t ntiles = (n + TILE - 1) / TILE;
    const uint32_t key_mask = (uint32_t)((uint64_t(1) << t.key_bits) - 1);
    uint32_t bad = 0, bad_key = 0;
    bool wide = false;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        uint32_t key[ITEMS];
        V val[ITEMS];
        const int64_t base = tile * TILE + (int64_t)w * ITEMS * WAVE;
        part_load(src, n, base, key, val, key_mask, bad, bad_key);
        probe_tile<MODE>(t, sp, out, parts, key, val, [&](int j) { return (uint32_t)(base + j * WAVE + l); }, wide, sm,
                         s_len);
    }
    part_finish<uint16_t, V, PART_BLOCK>(out, parts, sm);
    if (__any(bad_key != 0 || wide) && l == 0) set_flag(flags, FLAG_KEY_RANGE);
    if (__any(bad != 0) && l == 0) set_flag(flags, FLAG_VALUE_RANGE);
}

// The probe over the fact partitions' chunk lists.  Work item: the next 64
// (48) chunks of a partition, a tile.  The items lie in partition order, and
// the blocks of one XCD (consecutive blocks go to the XCDs in turn) take one
// eighth of them, so that an XCD works on one or two partitions at a time and
// their table slices stay in its L2.  Bound by the random reads of the table:
// at 60M rows it takes 444 us, 269 with the entries left unread, the gather
// costing about 2.3 clocks per lane and CU however it is issued (cached or not,
// ahead of time or not).  It takes the place of a second pass over the fact
// rows, the count, the expansion and the pass over its output: 1000 us.
template <class V, int MODE>
__global__ void __launch_bounds__(PART_BLOCK, PART_WAVES)
k_probe_chunks(Chunks<uint32_t, V> fact, int fact_parts, JoinTable t, Spill sp, Chunks<uint16_t, V> out, int parts,
               uint32_t* flags) {
    constexpr int ITEMS = PartItems<V>::value, W = PART_BLOCK / WAVE, PER = CHUNK / WAVE;
    constexpr int CPW = ITEMS / PER, CPT = W * CPW;   // chunks per wave and per tile
    static_assert(CPT == probe_chunks<V>(), "the grid's bound");
    __shared__ PartSmem<V> sm;
    __shared__ uint32_t s_item[PART_MAX + 1];         // first item of each partition
    __shared__ uint32_t s_len[W];
    const uint32_t lists = MODE == PROBE_ANY ? 0 : *t.list_n;
    const int tid = threadIdx.x, w = wave_index(), l = lane_id();
    part_init<uint16_t, V, PART_BLOCK>(sm);
    {
        const uint32_t nc = tid < fact_parts ? fact.dcount[tid] : 0;
        uint32_t tot;
        const uint32_t excl = block_excl_sum<PART_BLOCK>((nc + CPT - 1) / CPT, sm.scratch, &tot);
        if (tid < fact_parts) s_item[tid] = excl;
        if (tid == 0) s_item[fact_parts] = tot;
        __syncthreads();
    }
    if (MODE != PROBE_ANY && (lists != 0) != (MODE == PROBE_LISTS)) return;
    const uint32_t items = s_item[fact_parts];
    const uint32_t x = blockIdx.x % XCDS, per_xcd = gridDim.x / XCDS;
    const uint32_t i0 = (uint32_t)((uint64_t)items * x / XCDS), i1 = (uint32_t)((uint64_t)items * (x + 1) / XCDS);
    bool wide = false;
    // the numbers and row counts of an item's chunks are read while the item
    // before it is partitioned
    uint32_t id[CPW], rows[CPW];
    auto find = [&](uint32_t it) {
        int lo = 0, hi = fact_parts;                  // last partition with s_item <= it
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_item[mid] <= it) lo = mid; else hi = mid;
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        const uint32_t c0 = __builtin_amdgcn_readfirstlane((it - s_item[lo]) * CPT) + w * CPW;
        const uint32_t nc = fact.dcount[lo];
        const uint32_t* dir = fact.list + fact.first[lo];
#pragma unroll
        for (int q = 0; q < CPW; ++q) id[q] = dir[c0 + q < nc ? c0 + q : 0];     // the partition has an item, so a chunk
#pragma unroll
        for (int q = 0; q < CPW; ++q) rows[q] = c0 + q < nc ? fact.rows[id[q]] : 0;
    };
    constexpr bool AHEAD = MODE != PROBE_LISTS;       // (no registers left to read ahead)
    uint32_t it = i0 + blockIdx.x / XCDS;
    if (AHEAD && it < i1) find(it);
    for (; it < i1; it += per_xcd) {
        if (!AHEAD) find(it);
        int ll = l;
        asm volatile("" : "+v"(ll));                  // opaque, as in part_tile_rows
        uint32_t key[ITEMS];
        V val[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {             // rows past the end: read (the chunk holds them), not used
            const int64_t at = (int64_t)__builtin_amdgcn_readfirstlane(id[j / PER]) * CHUNK;
            // (read once: not kept in the L2, which holds the table's slice)
            key[j] = __builtin_nontemporal_load(&(fact.keys + at)[(j % PER) * WAVE + ll]);
            val[j] = __builtin_nontemporal_load(&(fact.vals + at)[(j % PER) * WAVE + ll]);
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if ((uint32_t)((j % PER) * WAVE + ll) >= rows[j / PER]) key[j] = PART_NONE;
        uint32_t at[CPW];
#pragma unroll
        for (int q = 0; q < CPW; ++q) at[q] = AHEAD ? id[q] : (uint32_t)__builtin_amdgcn_readfirstlane(id[q]);
        if (AHEAD && it + per_xcd < i1) find(it + per_xcd);
        probe_tile<MODE>(t, sp, out, parts, key, val,
                                           [&](int j) { return at[j / PER] * CHUNK + (j % PER) * WAVE + ll; }, wide, sm,
                                           s_len);
    }
    part_finish<uint16_t, V, PART_BLOCK>(out, parts, sm);
    if (__any(wide) && l == 0) set_flag(flags, FLAG_KEY_RANGE);
}

// The rows set aside, with every entry of their lists: the lists of 4096
// (2048) rows laid end to end, every thread finding the row and entry of its
// places.  (With 512 rows, lists of two entries filled an eighth of a tile.)
// Row of a set-aside place: of the source, or of the fact partitions' chunks.
template <class V, class Src>
struct PlaceCols {
    Src src;
    __device__ uint32_t key(uint32_t at) const {
        uint32_t k;
        V v;
        src.load(at, k, v);
        return k;
    }
    __device__ V value(uint32_t at) const {
        uint32_t k;
        V v;
        src.load(at, k, v);
        return v;
    }
};
template <class V>
struct PlaceChunks {
    const uint32_t* keys;
    const V* vals;
    __device__ uint32_t key(uint32_t at) const { return keys[at]; }
    __device__ V value(uint32_t at) const { return vals[at]; }
};
constexpr int LISTS_BLOCK = 1024;      // its LDS leaves one block per CU
template <class V, class Place>
__global__ void __launch_bounds__(LISTS_BLOCK)
k_probe_lists(Place place, JoinTable t, Spill sp, Chunks<uint16_t, V> out, int parts, uint32_t* flags) {
    constexpr int ITEMS = PartSmem<V, LISTS_BLOCK>::ITEMS, TILE = LISTS_BLOCK * ITEMS;
    constexpr int ROWS = sizeof(V) <= 4 ? 4096 : 2048, PER = ROWS / LISTS_BLOCK;
    __shared__ PartSmem<V, LISTS_BLOCK> sm;
    __shared__ int64_t s_first[ROWS];         // first place of each row's list
    __shared__ uint32_t s_list[ROWS];
    __shared__ V s_val[ROWS];
    __shared__ int64_t s_scan[LISTS_BLOCK / WAVE];
    const int tid = threadIdx.x, w = wave_index(), l = lane_id();
    const int64_t n = (int64_t)*sp.n;
    if ((int64_t)blockIdx.x * ROWS >= n) return;
    part_reopen<uint16_t, V, LISTS_BLOCK>(out, parts, sm);
    bool wide = false, room = true;
    for (int64_t r0 = (int64_t)blockIdx.x * ROWS; r0 < n; r0 += (int64_t)gridDim.x * ROWS) {
        __syncthreads();                              // the previous rows are expanded
        int64_t len[PER], mine = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {               // rows past the end: no entries
            const int64_t r = r0 + tid * PER + q;
            const uint32_t at = sp.at[r < n ? r : n - 1];
            const uint32_t list = t.slot[place.key(at)] & ~TJ_LIST;
            s_list[tid * PER + q] = list;
            s_val[tid * PER + q] = place.value(at);
            len[q] = t.list[list];
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (r0 + tid * PER + q >= n) len[q] = 0;
            mine += len[q];
        }
        int64_t total, at = block_excl_sum<LISTS_BLOCK>(mine, s_scan, &total);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            s_first[tid * PER + q] = at;
            at += len[q];
        }
        __syncthreads();
        int64_t q0 = 0;
        for (; room && q0 < total; q0 += TILE) {
            uint32_t key[ITEMS];
            V val[ITEMS];
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const int64_t q = q0 + (int64_t)w * ITEMS * WAVE + j * WAVE + l;
                const int64_t qc = q < total ? q : total - 1;
                int lo = 0;                   // last row whose list starts at or before q
#pragma unroll
                for (int step = ROWS / 2; step; step /= 2)
                    if (s_first[lo + step] <= qc) lo += step;
                uint32_t e = t.list[s_list[lo] + 1 + (uint32_t)(qc - s_first[lo])];
                if (q >= total) e = 0;
                wide |= (e & TJ_WIDE) != 0;
                key[j] = (e & ~TJ_WIDE) - 1;          // past the end: PART_NONE
                val[j] = s_val[lo];
            }
            room = part_tile_rows<uint16_t, V, LISTS_BLOCK>(out, parts, key, val, sm);
        }
        // pairs past the capacity are counted, not walked through: a key that
        // is frequent on both sides has more of them than a launch could
        if (tid == 0 && q0 < total) sm.over += (uint64_t)(total - q0);
    }
    part_finish<uint16_t, V, LISTS_BLOCK>(out, parts, sm);
    if (__any(wide) && l == 0) set_flag(flags, FLAG_KEY_RANGE);
}

// The fact partition (when there is one).
template <class V, class Src>
tqp_status table_partition(tqp_ctx* ctx, hipStream_t s, const TableJoin<V>& j, const Src& src, int64_t n_fact,
                           const char* name) {
    if (!j.fact_bits) return TQP_OK;
    return part_launch<uint32_t, V>(ctx, s, name, src, n_fact, j.fact, key_mask_for(j.t.key_bits), "part_list");
}

// The probe, after the table is built: j.grp holds the joined rows, by
// group partition.
template <class V, class Src>
tqp_status table_probe(tqp_ctx* ctx, hipStream_t s, const TableJoin<V>& j, const Src& src, int64_t n_fact,
                       const char* name, const char* short_name, const char* lists_name) {
    const int parts = 1 << j.grp.part_bits;
    if (n_fact > 0) {
        auto probe = [&](auto mode, const char* label) -> tqp_status {
            constexpr int MODE = decltype(mode)::value;
            if (j.fact_bits)
                TQP_LAUNCH(ctx, s, label,
                           (k_probe_chunks<V, MODE><<<(unsigned)j.grp.nblocks, PART_BLOCK, 0, s>>>(
                               j.fact, 1 << j.fact_bits, j.t, j.spill, j.grp, parts, ctx->d_err)));
            else
                TQP_LAUNCH(ctx, s, label,
                           (k_probe_cols<V, Src, MODE><<<(unsigned)j.grp.nblocks, PART_BLOCK, 0, s>>>(
                               src, j.t, j.spill, j.grp, parts, ctx->d_err)));
            return TQP_OK;
        };
        tqp_status st;
        if (n_fact < TJ_SHORT_ROWS) {
            if ((st = probe(std::integral_constant<int, PROBE_ANY>{}, name)) != TQP_OK) return st;
        } else {
            if ((st = probe(std::integral_constant<int, PROBE_UNIQUE>{}, name)) != TQP_OK) return st;
            if ((st = probe(std::integral_constant<int, PROBE_LISTS>{}, short_name)) != TQP_OK) return st;
        }
        if (j.fact_bits) {
            using Place = PlaceChunks<V>;
            TQP_LAUNCH(ctx, s, lists_name,
                       (k_probe_lists<V, Place><<<(unsigned)j.dup_blocks, LISTS_BLOCK, 0, s>>>(
                           Place{j.fact.keys, j.fact.vals}, j.t, j.spill, j.grp, parts, ctx->d_err)));
        } else {
            using Place = PlaceCols<V, Src>;
            TQP_LAUNCH(ctx, s, lists_name,
                       (k_probe_lists<V, Place><<<(unsigned)j.dup_blocks, LISTS_BLOCK, 0, s>>>(
                           Place{src}, j.t, j.spill, j.grp, parts, ctx->d_err)));
        }
    }
    return chunks_list(ctx, s, "group_list", j.grp);
}

}  // namespace tqp
