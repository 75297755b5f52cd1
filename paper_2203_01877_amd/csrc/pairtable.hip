// The join of pairs by a key table (pairtable.hpp): its rule, and the kernels
// that do not depend on the source of the rows.
#include "pairtable.hpp"

namespace tqp {

constexpr int PLACES_ITEMS = 8;

// Keys with several rows: a place in the list, its blocks' order not kept.
__global__ void __launch_bounds__(PAIR_BLOCK) k_pair_places(PairTable t) {
    __shared__ uint32_t s_scan[PAIR_BLOCK / WAVE];
    __shared__ uint32_t s_base;
    const int tid = threadIdx.x;
    const int64_t n = int64_t(1) << t.key_bits;
    const int64_t base = (int64_t)blockIdx.x * PAIR_BLOCK * PLACES_ITEMS;
    uint32_t cnt[PLACES_ITEMS], mine = 0;
#pragma unroll
    for (int j = 0; j < PLACES_ITEMS; ++j) {
        const int64_t k = base + j * PAIR_BLOCK + tid;
        cnt[j] = t.slot[k < n ? k : n - 1].cnt;
        if (k >= n || cnt[j] < 2) cnt[j] = 0;
        mine += cnt[j];
    }
    uint32_t total;
    uint32_t at = block_excl_sum<PAIR_BLOCK>(mine, s_scan, &total);
    if (total == 0) return;
    if (tid == 0) s_base = atomicAdd(t.list_n, total);
    __syncthreads();
    at += s_base;
#pragma unroll
    for (int j = 0; j < PLACES_ITEMS; ++j) {
        if (cnt[j] == 0) continue;
        t.slot[base + j * PAIR_BLOCK + tid].at = at;
        at += cnt[j];
    }
}

// The pairs of the fact rows with long lists: a block per row.
__global__ void __launch_bounds__(PAIR_BLOCK) k_pair_long(PairTable t, int32_t* out_l, int32_t* out_r, int64_t cap) {
    const uint32_t n = *t.span_n;
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        const PairSpan p = t.span[i];
        const PairSlot s = t.slot[p.key];
        const int64_t left = cap - p.out;
        const uint32_t cnt = left < s.cnt ? (uint32_t)left : s.cnt;
#pragma unroll 4
        for (uint32_t q = threadIdx.x; q < cnt; q += PAIR_BLOCK) {
            out_l[(int64_t)p.out + q] = (int32_t)p.l;
            out_r[(int64_t)p.out + q] = (int32_t)t.list[s.at + q];
        }
    }
}

// The slots of 2^20 keys (8 MB) are about what an XCD's L2 still serves in part;
// beyond it every row's slot is a read from the last-level cache, about 50 per
// nanosecond, which is what the sorts cost.  Clearing and scanning the slots must
// not outweigh the rows.  6M x 150k rows (2^18 keys) in all: 217 us, 354 by the
// sorts.  A digit width set by the caller asks for the sorts.
constexpr int PAIR_MAX_KEY_BITS = 20;
bool pair_table_ok(const tqp_ctx* ctx, int64_t n_fact, int64_t n_dim, int key_bits) {
    if (ctx->digit_bits != 8) return false;
    return key_bits <= PAIR_MAX_KEY_BITS && (int64_t(1) << key_bits) <= 8 * (n_fact + n_dim);
}

tqp_status pair_places(tqp_ctx* ctx, hipStream_t s, const PairTable& t) {
    TQP_LAUNCH(ctx, s, "fragment_pair_places",
               (k_pair_places<<<grid_for(int64_t(1) << t.key_bits, PAIR_BLOCK * PLACES_ITEMS, 0), PAIR_BLOCK, 0, s>>>(t)));
    return TQP_OK;
}
tqp_status pair_long(tqp_ctx* ctx, hipStream_t s, const PairTable& t, int32_t* out_l, int32_t* out_r, int64_t cap) {
    TQP_LAUNCH(ctx, s, "fragment_pairs_long",
               (k_pair_long<<<(unsigned)ctx->num_cus * 4, PAIR_BLOCK, 0, s>>>(t, out_l, out_r, cap)));
    return TQP_OK;
}

}  // namespace tqp
