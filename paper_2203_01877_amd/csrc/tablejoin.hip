// The rule of the join by a key table (tablejoin.hpp).
#include "tablejoin.hpp"

namespace tqp {

__global__ void __launch_bounds__(LIST_BLOCK)
k_chunks_list(const uint8_t* label, const uint64_t* pool, const uint32_t* dcount, uint32_t* cursor, uint32_t* list,
              uint32_t* first, int parts, int64_t nchunk) {
    __shared__ uint32_t s_cnt[PART_MAX], s_at[PART_MAX];
    __shared__ uint32_t s_scan[LIST_BLOCK / WAVE];
    const int tid = threadIdx.x;
    static_assert(LIST_BLOCK == PART_MAX, "one thread per partition");
    s_cnt[tid] = 0;
    uint32_t tot;
    const uint32_t f = block_excl_sum<LIST_BLOCK>(tid < parts ? dcount[tid] : 0, s_scan, &tot);
    if (blockIdx.x == 0 && tid < parts) first[tid] = f;
    // chunks are claimed in order, each by one tile; those past the pool's end
    // were neither labelled nor counted
    int64_t n = (int64_t)(*pool >> POOL_ROW_BITS);
    if (n > nchunk) n = nchunk;
    const int64_t i0 = ((int64_t)blockIdx.x * LIST_BLOCK + tid) * LIST_ITEMS;
    uint32_t d[LIST_ITEMS];
    if (i0 + LIST_ITEMS <= n) {
        static_assert(LIST_ITEMS == 16, "one 16-byte load");
        const uint4 v = *reinterpret_cast<const uint4*>(label + i0);       // label is 256-byte aligned
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < LIST_ITEMS; ++j) d[j] = w[j / 4] >> (8 * (j % 4)) & 0xFF;
    } else {
#pragma unroll
        for (int j = 0; j < LIST_ITEMS; ++j) d[j] = i0 + j < n ? label[i0 + j] : PART_MAX;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LIST_ITEMS; ++j)
        if (d[j] < (uint32_t)parts) atomicAdd(&s_cnt[d[j]], 1u);
    __syncthreads();
    s_at[tid] = tid < parts && s_cnt[tid] ? f + atomicAdd(&cursor[tid], s_cnt[tid]) : 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LIST_ITEMS; ++j)
        if (d[j] < (uint32_t)parts) list[atomicAdd(&s_at[d[j]], 1u)] = (uint32_t)(i0 + j);
}

// The table needs a slot per key value and the group partitions at most 2^13
// LDS slots each (21 bits in 256 partitions); beyond 2^28 keys, or eight keys
// per row, clearing and reading slots without rows outweighs the passes saved.
// At 60k x 15k rows it takes 79 us where the sorts take 152, at 3M x 750k 100
// against 220, at 60M x 15M 1258 against 1857; with every key on two dim rows 327
// against 459 at 6M x 1.5M and 1681 against 1733 at 40M x 10M, on eight 660 against
// 1430; near the limits (where only a join capacity of several times the fact
// rows gives the sorts as much scratch) 27M x 6.75M rows over 2^28 keys 1081
// against 1501, 3.4M x 850k over 2^25 348 against 367.  A digit width set by the
// caller asks for the sorts.
bool table_join_ok(const tqp_ctx* ctx, int64_t n_fact, int64_t n_dim, int key_bits, int group_bits) {
    if (ctx->digit_bits != 8) return false;
    if (key_bits > TJ_MAX_KEY_BITS || group_bits > TJ_MAX_GROUP_BITS) return false;
    return (int64_t(1) << key_bits) <= 8 * (n_fact + n_dim);
}

}  // namespace tqp
