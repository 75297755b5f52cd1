// Equi-join by a table over the key domain that yields (fact row, dim row)
// pairs in about the order of the fact rows, for consumers that read both
// sides' columns through the pairs and do not depend on their order: the fact
// columns are then read in one forward sweep, where the pairs of the sort-based
// join come in key order and read them at random.
//
//   count    per key, the kept dim rows: their number and one of them
//   places   keys with several rows get a place in the list of dim rows
//   lists    those rows enter it (nothing to do while keys are unique)
//   probe    every kept fact row reads its key's slot and writes its pairs; a
//            tile claims its output with one atomic.  Rows with long lists
//            only reserve their output, and a last kernel writes it.
#pragma once

#include "dev.hpp"
#include "host.hpp"
#include "radix.hpp"

namespace tqp {

// A key's slot: dim rows with it, and the one (or the start of their list).
struct alignas(8) PairSlot {
    uint32_t cnt;
    uint32_t at;
};
// Output reserved by a fact row with a long list.
struct PairSpan {
    uint32_t out, l, key;
};

struct PairTable {
    PairSlot* slot = nullptr;          // [2^key_bits] (zero on entry)
    uint32_t* rank = nullptr;          // [n_dim] number of each row among its key's
    uint32_t* list = nullptr;          // [n_dim]
    uint32_t* list_n = nullptr;        // list places taken (zero on entry)
    PairSpan* span = nullptr;          // [cap / PAIR_LONG + 1]
    uint32_t* span_n = nullptr;        // (zero on entry)
    int key_bits = 0;
};

constexpr int PAIR_BLOCK = 256;
constexpr int PROBE_BLOCK = 512, PROBE_ITEMS = 8;        // a probe tile: 4096 rows
constexpr uint32_t PAIR_LONG = 64;     // a list longer than this is left to k_pair_long

inline void pair_table_reserve(Arena& a, PairTable& t, int64_t n_dim, int key_bits, int64_t cap) {
    t.key_bits = key_bits;
    t.slot = a.zero<PairSlot>(int64_t(1) << key_bits);
    t.list_n = a.zero<uint32_t>(1);
    t.span_n = a.zero<uint32_t>(1);
    t.rank = a.scratch<uint32_t>(n_dim);
    t.list = a.scratch<uint32_t>(n_dim);
    t.span = a.scratch<PairSpan>(cap / PAIR_LONG + 1);
}

// Rows of a source whose key lies in the table's domain; the others are
// flagged when the source keeps them.
template <class Src>
__device__ __forceinline__ bool pair_key(const Src& src, const PairTable& t, int64_t i, uint32_t& k, bool& bad) {
    const bool keep = src.load_key(i, k);
    const bool in = (uint64_t)k >> t.key_bits == 0;
    bad |= keep && !in;
    return keep && in;
}

// Rows of one key are counted once per wave (wave_match): 900k dim rows, half of
// them with one key, 352 us; by an atomic per row 5582.
template <class Src>
__global__ void __launch_bounds__(PAIR_BLOCK)
k_pair_count(Src src, PairTable t, uint32_t* flags) {
    __shared__ WaveMatch s_match[PAIR_BLOCK / WAVE];
    WaveMatch& match = s_match[threadIdx.x / WAVE];
    const int64_t n = src.size();
    bool bad = false;
    for (int64_t i0 = (int64_t)blockIdx.x * PAIR_BLOCK; i0 < n; i0 += (int64_t)gridDim.x * PAIR_BLOCK) {
        const int64_t i = i0 + threadIdx.x;
        uint32_t k = 0;
        const bool live = i < n && pair_key(src, t, i, k, bad);
        int leader;
        uint32_t rank, count, base = 0;
        wave_match(match, k, live, leader, rank, count);
        if (live && leader == lane_id()) {
            base = atomicAdd(&t.slot[k].cnt, count);
            t.slot[k].at = (uint32_t)i;               // the row, while it is the only one
        }
        base = wave_shfl(base, leader);
        if (live) t.rank[i] = base + rank;
    }
    if (bad) set_flag(flags, FLAG_KEY_RANGE);
}

__global__ void k_pair_places(PairTable t);

template <class Src>
__global__ void __launch_bounds__(PAIR_BLOCK)
k_pair_lists(Src src, PairTable t) {
    if (*t.list_n == 0) return;
    const int64_t n = src.size();
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * PAIR_BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * PAIR_BLOCK) {
        uint32_t k;
        if (!pair_key(src, t, i, k, bad)) continue;
        const PairSlot s = t.slot[k];
        if (s.cnt > 1) t.list[s.at + t.rank[i]] = (uint32_t)i;
    }
}

// One tile per block, all its slots read at once.  Bound by the latency of the
// slot reads (from L2) and by the tiles' claims, which meet at one word (about
// 50 per microsecond): 6M rows, 1.1M pairs take 39 us in tiles of 4096 rows, 45
// in tiles of 8192, 53 to 57 in tiles of 8192 to 16384 with 16 rows per thread.
// The sorts of both sides and the join they replace took 200.
template <class Src>
__global__ void __launch_bounds__(PROBE_BLOCK)
k_pair_probe(Src src, PairTable t, int32_t* out_l, int32_t* out_r, int64_t cap, int64_t* d_n, uint32_t* flags) {
    constexpr int W = PROBE_BLOCK / WAVE, COUNTS = PROBE_ITEMS * W, PER = COUNTS / WAVE;
    static_assert(COUNTS % WAVE == 0, "counts per lane");
    __shared__ int64_t s_at[COUNTS];                  // pairs of each (item, wave), then where they go
    const int tid = threadIdx.x, w = tid / WAVE, l = lane_id();
    const int64_t n = src.size();
    const int64_t base = (int64_t)blockIdx.x * (PROBE_BLOCK * PROBE_ITEMS);
    uint32_t key[PROBE_ITEMS];
    bool live[PROBE_ITEMS], bad = false;
#pragma unroll
    for (int j = 0; j < PROBE_ITEMS; ++j) {            // rows past the end: the last one, not used
        const int64_t i = base + j * PROBE_BLOCK + tid;
        live[j] = src.load_key(i < n ? i : n - 1, key[j]) && i < n;
    }
    PairSlot s[PROBE_ITEMS];
#pragma unroll
    for (int j = 0; j < PROBE_ITEMS; ++j) {
        const bool in = (uint64_t)key[j] >> t.key_bits == 0;
        bad |= live[j] && !in;
        live[j] = live[j] && in;
        s[j] = t.slot[live[j] ? key[j] : 0];
    }
    uint64_t before[PROBE_ITEMS];                      // pairs of the wave's lanes before this one
#pragma unroll
    for (int j = 0; j < PROBE_ITEMS; ++j) {
        if (!live[j]) s[j].cnt = 0;
        int64_t total;
        if (__any(s[j].cnt > 1)) {
            const int64_t incl = wave_incl_sum((int64_t)s[j].cnt);
            before[j] = (uint64_t)(incl - s[j].cnt);
            total = wave_read(incl, WAVE - 1);
        } else {
            const uint64_t m = __ballot(s[j].cnt != 0);
            before[j] = __popcll(m & ((uint64_t(1) << l) - 1));
            total = __popcll(m);
        }
        if (l == 0) s_at[j * W + w] = total;
    }
    __syncthreads();
    if (w == 0) {
        int64_t c[PER], mine = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) mine += c[q] = s_at[l * PER + q];
        const int64_t incl = wave_incl_sum(mine), total = wave_read(incl, WAVE - 1);
        int64_t at = 0;
        if (l == 0 && total)
            at = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(d_n), (unsigned long long)total);
        at = wave_read(at, 0);
        if (l == 0 && total && at + total > cap) set_flag(flags, FLAG_CAPACITY);
        at += incl - mine;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            s_at[l * PER + q] = at;
            at += c[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PROBE_ITEMS; ++j) {
        if (s[j].cnt == 0) continue;
        const int32_t row = (int32_t)(base + j * PROBE_BLOCK + tid);
        const int64_t o = s_at[j * W + w] + (int64_t)before[j];
        if (o >= cap) continue;
        if (s[j].cnt == 1) {
            out_l[o] = row;
            out_r[o] = (int32_t)s[j].at;
        } else if (s[j].cnt <= PAIR_LONG) {
            for (uint32_t q = 0; q < s[j].cnt && o + q < cap; ++q) {
                out_l[o + q] = row;
                out_r[o + q] = (int32_t)t.list[s[j].at + q];
            }
        } else {
            // spans begin below cap and are longer than PAIR_LONG: they fit
            t.span[atomicAdd(t.span_n, 1u)] = PairSpan{(uint32_t)o, (uint32_t)row, key[j]};
        }
    }
    if (__any(bad) && l == 0) set_flag(flags, FLAG_KEY_RANGE);
}

__global__ void k_pair_long(PairTable t, int32_t* out_l, int32_t* out_r, int64_t cap);

// Whether a join takes the table, and its launches (pairtable.hip holds the rule).
bool pair_table_ok(const tqp_ctx* ctx, int64_t n_fact, int64_t n_dim, int key_bits);
tqp_status pair_places(tqp_ctx* ctx, hipStream_t s, const PairTable& t);
tqp_status pair_long(tqp_ctx* ctx, hipStream_t s, const PairTable& t, int32_t* out_l, int32_t* out_r, int64_t cap);

template <class Src>
tqp_status pair_build(tqp_ctx* ctx, hipStream_t s, const PairTable& t, const Src& dim, int64_t n_dim) {
    if (n_dim == 0) return TQP_OK;
    const int grid = grid_for(n_dim, PAIR_BLOCK, (int64_t)ctx->num_cus * 8);
    TQP_LAUNCH(ctx, s, "fragment_pair_count", (k_pair_count<Src><<<grid, PAIR_BLOCK, 0, s>>>(dim, t, ctx->d_err)));
    const tqp_status st = pair_places(ctx, s, t);
    if (st != TQP_OK) return st;
    TQP_LAUNCH(ctx, s, "fragment_pair_lists", (k_pair_lists<Src><<<grid, PAIR_BLOCK, 0, s>>>(dim, t)));
    return TQP_OK;
}

template <class Src>
tqp_status pair_probe(tqp_ctx* ctx, hipStream_t s, const PairTable& t, const Src& fact, int64_t n_fact, int32_t* out_l,
                      int32_t* out_r, int64_t cap, int64_t* d_n) {
    if (n_fact == 0) return TQP_OK;
    TQP_LAUNCH(ctx, s, "fragment_pairs",
               (k_pair_probe<Src><<<grid_for(n_fact, PROBE_BLOCK * PROBE_ITEMS, 0), PROBE_BLOCK, 0, s>>>(
                   fact, t, out_l, out_r, cap, d_n, ctx->d_err)));
    return pair_long(ctx, s, t, out_l, out_r, cap);
}

}  // namespace tqp
