// Filter (Section 3.1): a conjunction of column-versus-constant comparisons
// evaluated per row, then stream compaction into a selection vector of row ids
// (the index form of the bitmap filter), with an optional carried column.
//
// Per tile: one ballot per 64 rows gives the wave's survivors and each lane's
// rank among them; a block scan and a decoupled look-back give the tile's
// output base.  The row count stays on the device (and the input's may come
// from the device: d_n).
#pragma once
#include "dev.hpp"
#include "host.hpp"
#include "radix.hpp"

namespace tqp {

constexpr int FILTER_MAX_PREDS = 4;

struct FilterPreds {
    const void* col[FILTER_MAX_PREDS];
    int32_t type[FILTER_MAX_PREDS];    // 1 = int8, 2 = int32, 3 = int64
    int32_t op[FILTER_MAX_PREDS];
    int64_t k[FILTER_MAX_PREDS];
    int32_t np;
    // ok[j] for rows idx[j] (already clamped into range): per predicate, the
    // column type is decided once and all the rows' values are loaded before
    // any is compared, so they are in flight together.
    template <int ITEMS>
    __device__ void eval(const int64_t (&idx)[ITEMS], bool (&ok)[ITEMS]) const {
        for (int p = 0; p < np; ++p) {
            int64_t x[ITEMS];
            if (type[p] == 1) {
                const int8_t* c = (const int8_t*)col[p];
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) x[j] = c[idx[j]];
            } else if (type[p] == 2) {
                const int32_t* c = (const int32_t*)col[p];
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) x[j] = c[idx[j]];
            } else {
                const int64_t* c = (const int64_t*)col[p];
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) x[j] = c[idx[j]];
            }
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) ok[j] = ok[j] & cmp_eval(x[j], op[p], k[p]);
        }
    }
};

// Bound by HBM: the predicate columns, the lines of the carried column that
// hold a kept row, and the outputs.  60M rows, a 4- and an 8-byte predicate
// column and a carried column, 16% kept (about 1.05 GB): 275 us, where tiles of
// one round took 325 and those with a branch around each carried value's read
// 372.
template <int BLOCK, int ITEMS, int ROUNDS>
__global__ void __launch_bounds__(BLOCK)
k_filter(FilterPreds fp, int64_t n, const int32_t* carry, int32_t* out_row, int32_t* out_carry,
         int64_t cap, int64_t* d_count, uint64_t* status, uint32_t* tile_counter, uint32_t* flags,
         const int64_t* d_n) {
    constexpr int W = BLOCK / WAVE, MASKS = ROUNDS * ITEMS;
    constexpr int64_t TILE = (int64_t)BLOCK * MASKS;
    __shared__ uint64_t s_mask[ROUNDS > 1 ? W : 1][MASKS];     // survivors of each 64 rows
    __shared__ int64_t s_wave[W];
    __shared__ int64_t s_base;
    __shared__ uint32_t s_tile;
    const int tid = threadIdx.x, w = tid / WAVE, l = lane_id();
    if (d_n) {                                 // rows counted on the device, at most n
        const int64_t t = *d_n;
        n = t < n ? t : n;
    }
    if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
    __syncthreads();
    const int64_t tile = s_tile;
    const int64_t ntiles = (n + TILE - 1) / TILE;
    if (tile >= ntiles) {
        if (ntiles == 0 && tile == 0 && tid == 0) *d_count = 0;
        return;
    }
    const int64_t chunk = tile * TILE + (int64_t)w * MASKS * WAVE;
    int64_t wc = 0;
    uint64_t mask[ITEMS];                      // of a single round (one in LDS cost a small filter 0.6 us)
#pragma unroll 1
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t r0 = chunk + (int64_t)r * ITEMS * WAVE;
        int64_t idx[ITEMS];
        bool ok[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int64_t i = r0 + j * WAVE + l;
            ok[j] = i < n;
            idx[j] = ok[j] ? i : n - 1;       // n >= 1: the tile exists
        }
        fp.eval<ITEMS>(idx, ok);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint64_t m = ballot(ok[j]);
            if constexpr (ROUNDS > 1) {
                if (l == 0) s_mask[w][r * ITEMS + j] = m;
            } else {
                mask[j] = m;
            }
            wc += popc64(m);
        }
    }
    if (l == 0) s_wave[w] = wc;
    __syncthreads();
    if (w == 0) {
        int64_t tot = 0;
        for (int ww = 0; ww < W; ++ww) tot += s_wave[ww];
        const int64_t base = lookback64(status, tile, tot, flags);
        if (tid == 0) {
            int64_t run = 0;
            for (int ww = 0; ww < W; ++ww) { const int64_t x = s_wave[ww]; s_wave[ww] = run; run += x; }
            s_base = base;
            if (tile == ntiles - 1) {
                *d_count = base + tot;
                if (base + tot > cap) set_flag(flags, FLAG_CAPACITY);
            }
        }
    }
    __syncthreads();
    int64_t pos = s_base + s_wave[w];
#pragma unroll 1
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t r0 = chunk + (int64_t)r * ITEMS * WAVE;
        int64_t o[ITEMS];                      // output position, -1: none
        int32_t c[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint64_t m = ROUNDS > 1 ? s_mask[ROUNDS > 1 ? w : 0][r * ITEMS + j] : mask[j];
            o[j] = pos + popc64(m & lanemask_lt());
            if (!((m >> l) & 1) || o[j] >= cap) o[j] = -1;
            pos += popc64(m);
        }
        if (out_carry) {
            // rows that are out read the tile's first row: no branch between the loads
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) c[j] = carry[o[j] >= 0 ? r0 + j * WAVE + l : tile * TILE];
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (o[j] >= 0) {
                out_row[o[j]] = (int32_t)(r0 + j * WAVE + l);
                if (out_carry) out_carry[o[j]] = c[j];
            }
        }
    }
}

constexpr int FILTER_BLOCK = 256, FILTER_ITEMS = 16;
constexpr int64_t FILTER_TILE = FILTER_BLOCK * FILTER_ITEMS;   // rows per look-back word

// Long tiles of four rounds from six short ones per CU on: scan and filter of
// 60M rows 686 us with long tiles against 732, of 16M 206 against 227, of 8M
// 115 against 129; of 4M 70 against 68 and of 1M 46 against 34, where the long
// tiles leave CUs without one.
constexpr int FILTER_ROUNDS = 4;
inline tqp_status filter_launch(tqp_ctx* ctx, hipStream_t s, const char* name, const FilterPreds& fp, int64_t n,
                                const int32_t* carry, int32_t* out_row, int32_t* out_carry, int64_t cap,
                                int64_t* d_count, uint64_t* status, uint32_t* counter, const int64_t* d_n = nullptr) {
    if (n > FILTER_TILE * 6 * ctx->num_cus)
        TQP_LAUNCH(ctx, s, name,
                   (k_filter<FILTER_BLOCK, FILTER_ITEMS, FILTER_ROUNDS>
                    <<<grid_for(n, FILTER_TILE * FILTER_ROUNDS, 0), FILTER_BLOCK, 0, s>>>(
                        fp, n, carry, out_row, out_carry, cap, d_count, status, counter, ctx->d_err, d_n)));
    else
        TQP_LAUNCH(ctx, s, name,
                   (k_filter<FILTER_BLOCK, FILTER_ITEMS, 1><<<grid_for(n, FILTER_TILE, 0), FILTER_BLOCK, 0, s>>>(
                       fp, n, carry, out_row, out_carry, cap, d_count, status, counter, ctx->d_err, d_n)));
    return TQP_OK;
}

}  // namespace tqp
