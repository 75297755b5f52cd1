// Flags fragments over a small join-key domain (see flags_direct.hpp).
#include "flags_direct.hpp"

namespace tqp {

namespace {

constexpr int BLOCK = 512;
constexpr int ITEMS = 4;
constexpr int LDS_KEYS_LOG2 = 12;                     // key domain that a fact block can count itself
constexpr int64_t LDS_DIM_ROWS = 4096;                // and the dim rows it then reads
constexpr int BLOCKS_PER_CU = 4;

// The table's rule: at most 2^26 keys, and no more than four per dim row (with
// 2^18 free), so that clearing and filling the table costs less than the dim
// sort it replaces (60k x 15M rows over 2^24 keys: 138 us against 277 with the
// sorts; 1k x 150k: 16 against 133; 60M x 1.5M: 550 against 1623).  The rule
// leaves the fact rows out: requests over row ranges of one table then all
// take the same form, whatever their size.  A digit width set by the caller
// asks for the sorts.  The free keys are the one case in which the table needs
// more scratch than the sorts, at most 1.1 MB of it: a caller's workspace that
// the sorts fit and the table does not is given to the sorts, and a batch's
// tables are bounded as a whole (FLAGS_BATCH_SPARE).
constexpr int MAX_KEY_BITS = 26;
constexpr int64_t FREE_KEYS = int64_t(1) << 18;

struct AccSmem {
    // a slot per lane, shared by the block's waves: no conflicts within a wave
    unsigned long long v[FLAGS_GROUPS * 3][WAVE];
    int64_t join[BLOCK / WAVE];
};

// Sums of fact rows [r0, r1) into the thread's slots; weight(k) = kept dim
// rows with key k.
template <class Weight>
__device__ __forceinline__ void sum_rows(const FlagsDirect& f, int64_t r0, int64_t r1, AccSmem& sm,
                                         const Weight& weight, uint32_t* flags, int64_t& joined) {
    const int tid = threadIdx.x, l = lane_id();
    uint32_t bad_key = 0, bad_val = 0;
    constexpr int64_t STEP = (int64_t)BLOCK * ITEMS;
    for (int64_t i0 = r0 + tid; i0 < r1; i0 += STEP) {
        uint32_t k[ITEMS];
        int32_t dt[ITEMS];
        uint32_t wt[ITEMS];
        bool any = false;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {             // clamped index: no branch between the loads
            const int64_t i = i0 + (int64_t)j * BLOCK;
            const int64_t ic = i < r1 ? i : r1 - 1;
            k[j] = (uint32_t)f.fk[ic];
            dt[j] = f.date[ic];
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const bool keep = i0 + (int64_t)j * BLOCK < r1 && dt[j] < f.D;
            const bool in = (k[j] & ~f.key_mask) == 0;
            bad_key |= (uint32_t)(keep & !in);
            wt[j] = weight(keep & in ? k[j] : 0u);    // rows that are out look up key 0: no branch
            if (!(keep & in)) wt[j] = 0;
            any |= wt[j] != 0;
        }
        if (!__any(any)) continue;
        // rows that do not count read the chunk's first row: one line for all
        // of them, and no branch between the loads
        int64_t pr[ITEMS], dc[ITEMS];
        int32_t fa[ITEMS], fb[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int64_t i = wt[j] ? i0 + (int64_t)j * BLOCK : r0;
            pr[j] = f.price[i];
            dc[j] = f.disc[i];
            fa[j] = f.flagA[i];
            fb[j] = f.flagB[i];
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (!wt[j]) continue;
            joined += wt[j];
            const bool ok = (unsigned)fa[j] <= 2u && (unsigned)fb[j] <= 1u;
            bad_val |= (uint32_t)!ok;
            if (!ok) continue;
            const int g = 3 * (fa[j] * 2 + fb[j]);
            const unsigned long long w = wt[j];
            atomicAdd(&sm.v[g][l], (unsigned long long)(pr[j] * (100 - dc[j])) * w);
            atomicAdd(&sm.v[g + 1][l], w);
            atomicAdd(&sm.v[g + 2][l], (unsigned long long)pr[j] * w);
        }
    }
    if (__any(bad_key != 0) && lane_id() == 0) set_flag(flags, FLAG_KEY_RANGE);
    if (__any(bad_val != 0) && lane_id() == 0) set_flag(flags, FLAG_VALUE_RANGE);
}

__device__ __forceinline__ void acc_init(AccSmem& sm) {
    for (int a = threadIdx.x; a < FLAGS_GROUPS * 3 * WAVE; a += BLOCK) (&sm.v[0][0])[a] = 0;
    __syncthreads();
}

// The block's sums to its slot of the fragment's partial array.
__device__ __forceinline__ void acc_flush(AccSmem& sm, int64_t joined, int64_t* part, int64_t nslot, int64_t slot) {
    const int w = threadIdx.x / WAVE, l = lane_id();
    const int64_t j = wave_sum(joined);
    if (l == 0) sm.join[w] = j;
    __syncthreads();
    for (int a = w; a < FLAGS_GROUPS * 3; a += BLOCK / WAVE) {
        const int64_t t = wave_sum((int64_t)sm.v[a][l]);
        if (l == 0) part[a * nslot + slot] = t;
    }
    if (threadIdx.x == 0) {
        int64_t t = 0;
#pragma unroll
        for (int q = 0; q < BLOCK / WAVE; ++q) t += sm.join[q];
        part[(FLAGS_PART - 1) * nslot + slot] = t;
    }
}

// Dim rows [r0, r1) that pass their predicate, entered into the table: rows of
// one key once per wave, and the word that says that keys repeat once per
// wave.  With an atomic per row the rows of a frequent key, and with a store
// per further row all of them, take turns on one word (4.6 ns each): 3M dim
// rows, half of them with one key, 20.3 ms and 0.27 so; every key twice 1.76 and
// 0.25; every key once 0.12 both ways.
__device__ __forceinline__ void enter_dim(const FlagsDirect& f, int64_t r0, int64_t r1, uint32_t* flags) {
    __shared__ WaveMatch s_match[BLOCK / WAVE];
    WaveMatch& match = s_match[threadIdx.x / WAVE];
    bool bad = false, again = false;
    for (int64_t i0 = r0; i0 < r1; i0 += BLOCK) {
        const int64_t i = i0 + threadIdx.x, ic = i < r1 ? i : r1 - 1;
        const uint32_t k = (uint32_t)f.pk[ic];
        const bool kept = i < r1 && f.seg[ic] == f.c, in = (k & ~f.key_mask) == 0;
        bad |= kept && !in;
        const bool live = kept && in;
        int leader;
        uint32_t rank, count;
        wave_match(match, k, live, leader, rank, count);
        if (live && leader == lane_id()) {
            const uint32_t bit = 1u << (k & 31);
            uint32_t* word = &f.bits[k >> 5];
            // (a frequent key's bit is mostly set by now)
            const uint32_t old = count > 1 && (ld_relaxed(word) & bit)
                                     ? bit
                                     : __hip_atomic_fetch_or(word, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t more = old & bit ? count : count - 1;
            if (more) {
                atomic_add(&f.extra[k], more);
                again = true;
            }
        }
    }
    if (__any(again) && lane_id() == 0 && ld_relaxed(f.repeats) == 0) st_relaxed(f.repeats, 1u);
    if (__any(bad) && lane_id() == 0) set_flag(flags, FLAG_KEY_RANGE);
}

__device__ __forceinline__ void table_rows(const FlagsDirect& f, int64_t r0, int64_t r1, int64_t slot, AccSmem& sm,
                                           uint32_t* flags) {
    acc_init(sm);
    int64_t joined = 0;
    const uint32_t* bits = f.bits;
    const uint32_t* extra = f.extra;
    if (*f.repeats == 0)
        sum_rows(f, r0, r1, sm, [&](uint32_t k) { return (bits[k >> 5] >> (k & 31)) & 1u; }, flags, joined);
    else
        sum_rows(f, r0, r1, sm,
                 [&](uint32_t k) {
                     const uint32_t b = (bits[k >> 5] >> (k & 31)) & 1u;
                     return b ? 1 + extra[k] : 0;
                 },
                 flags, joined);
    acc_flush(sm, joined, f.part, f.nslot, slot);
}

__global__ void __launch_bounds__(BLOCK) k_flags_dim(FlagsDirect f, uint32_t* flags) {
    const int64_t per = (f.n_dim + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = blockIdx.x * per;
    enter_dim(f, r0, r0 + per < f.n_dim ? r0 + per : f.n_dim, flags);
}

__device__ __forceinline__ void block_rows(int64_t n, int64_t& r0, int64_t& r1) {
    int64_t per = (n + gridDim.x - 1) / gridDim.x;
    per = (per + WAVE - 1) / WAVE * WAVE;
    r0 = blockIdx.x * per;
    r1 = r0 + per < n ? r0 + per : n;
    if (r0 > r1) r0 = r1;
}

// Bound by the fact columns' bytes: 8 B per row and the 18 B of rows whose
// lines hold a row that counts (with 19% of the rows counting, nearly every
// line).  6M x 150k rows: 29 us of 156 MB, where the sorts and the join took
// 207 (the join's reads through row ids alone 100).  Loads of the next round
// ahead, 2 or 8 rows per thread and non-temporal loads were no faster.
__global__ void __launch_bounds__(BLOCK) k_flags_fact(FlagsDirect f, uint32_t* flags) {
    __shared__ AccSmem sm;
    int64_t r0, r1;
    block_rows(f.n_fact, r0, r1);
    table_rows(f, r0, r1, blockIdx.x, sm, flags);
}

// A dim side of a few thousand rows over a few thousand keys: every block
// counts it in LDS, so that a small fragment is two launches (160k x 4096
// rows: 11 us, where the table's four launches take 17).
__global__ void __launch_bounds__(BLOCK) k_flags_fact_lds(FlagsDirect f, uint32_t* flags) {
    __shared__ AccSmem sm;
    __shared__ uint32_t s_cnt[1 << LDS_KEYS_LOG2];
    acc_init(sm);
    for (int i = threadIdx.x; i <= (int)f.key_mask; i += BLOCK) s_cnt[i] = 0;
    __syncthreads();
    uint32_t bad = 0;
    for (int64_t i0 = threadIdx.x; i0 < f.n_dim; i0 += BLOCK * ITEMS) {
        uint32_t k[ITEMS];
        int32_t sg[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int64_t i = i0 + j * BLOCK < f.n_dim ? i0 + j * BLOCK : f.n_dim - 1;
            k[j] = (uint32_t)f.pk[i];
            sg[j] = f.seg[i];
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (i0 + j * BLOCK >= f.n_dim || sg[j] != f.c) continue;
            if (k[j] & ~f.key_mask) bad = 1;
            else atomicAdd(&s_cnt[k[j]], 1u);
        }
    }
    if (blockIdx.x == 0 && __any(bad != 0) && lane_id() == 0) set_flag(flags, FLAG_KEY_RANGE);
    __syncthreads();
    int64_t r0, r1, joined = 0;
    block_rows(f.n_fact, r0, r1);
    sum_rows(f, r0, r1, sm, [&](uint32_t k) { return s_cnt[k]; }, flags, joined);
    acc_flush(sm, joined, f.part, f.nslot, blockIdx.x);
}

// Block sums of one fragment to its groups, in ascending packed-key order,
// skipping keys no row reached.
constexpr int FINAL_BLOCK = 1024;
__device__ __forceinline__ void finalize(const FlagsDirect& f) {
    __shared__ int64_t s_tot[FLAGS_PART];
    const int w = threadIdx.x / WAVE, l = lane_id();
    for (int a = w; a < FLAGS_PART; a += FINAL_BLOCK / WAVE) {
        constexpr int U = 8;                          // loads in flight per lane
        const int64_t n = f.nslot;
        int64_t t = 0;
        for (int64_t i0 = l; i0 < n; i0 += WAVE * U) {
            int64_t x[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int64_t i = i0 + j * WAVE;
                x[j] = f.part[a * n + (i < n ? i : n - 1)];
            }
#pragma unroll
            for (int j = 0; j < U; ++j) t += i0 + j * WAVE < n ? x[j] : 0;
        }
        t = wave_sum(t);
        if (l == 0) s_tot[a] = t;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int64_t g = 0;
    for (int k = 0; k < FLAGS_GROUPS; ++k) {
        const int64_t s = s_tot[k * 3], c = s_tot[k * 3 + 1], p = s_tot[k * 3 + 2];
        if (c == 0) continue;
        f.out.key[g] = k;
        f.out.sum[g] = s;
        f.out.cnt[g] = c;
        f.out.avg[g] = (double)p / (double)c;
        ++g;
    }
    *f.out.d_ngroups = g;
    if (f.out.d_join) *f.out.d_join = s_tot[FLAGS_PART - 1];
}

__global__ void __launch_bounds__(FINAL_BLOCK) k_flags_direct_final(FlagsDirect f) { finalize(f); }

// Batch forms: one block per work item.
__global__ void __launch_bounds__(BLOCK) k_batch_flags_dim(const FlagsDirect* frags, const FlagsItem* items,
                                                           uint32_t* flags) {
    const FlagsItem it = items[blockIdx.x];
    enter_dim(frags[it.frag], it.r0, it.r1, flags);
}
__global__ void __launch_bounds__(BLOCK) k_batch_flags_fact(const FlagsDirect* frags, const FlagsItem* items,
                                                            uint32_t* flags) {
    __shared__ AccSmem sm;
    const FlagsItem it = items[blockIdx.x];
    const FlagsDirect f = frags[it.frag];
    table_rows(f, it.r0, it.r1, it.slot, sm, flags);
}
__global__ void __launch_bounds__(FINAL_BLOCK) k_batch_flags_final(const FlagsDirect* frags) {
    finalize(frags[blockIdx.x]);
}

}  // namespace

bool flags_direct_ok(const tqp_ctx* ctx, const tqp_flags_fragment& f) {
    if (ctx->digit_bits != 8) return false;
    const int kb = norm_key_bits(f.key_bits);
    return kb <= MAX_KEY_BITS && (int64_t(1) << kb) <= 4 * f.n_dim + FREE_KEYS;
}

bool flags_direct_lds(const tqp_flags_fragment& f) {
    return norm_key_bits(f.key_bits) <= LDS_KEYS_LOG2 && f.n_dim <= LDS_DIM_ROWS;
}

int64_t flags_direct_words(const tqp_flags_fragment& f) {
    return ((int64_t(1) << norm_key_bits(f.key_bits)) + 31) / 32;
}

void flags_direct_fill(const tqp_flags_fragment& f, const tqp_flags_out& o, FlagsDirect& d) {
    d.fk = f.fk + f.row0;
    d.date = f.date + f.row0;
    d.price = f.price + f.row0;
    d.disc = f.disc + f.row0;
    d.flagA = f.flagA + f.row0;
    d.flagB = f.flagB + f.row0;
    d.n_fact = f.n_fact;
    d.pk = f.pk;
    d.seg = f.seg;
    d.n_dim = f.n_dim;
    d.D = f.D;
    d.c = f.c;
    d.key_mask = key_mask_for(norm_key_bits(f.key_bits));
    d.out = o;
}

tqp_status flags_direct_run(tqp_ctx* ctx, const tqp_flags_fragment& f, const tqp_flags_out& o, void* ws,
                            size_t* ws_bytes, hipStream_t s) {
    const bool lds = flags_direct_lds(f);
    FlagsDirect d{};
    flags_direct_fill(f, o, d);
    // one row per thread while that does not fill the chip, then a few
    // resident blocks per CU
    d.nslot = grid_for(f.n_fact, BLOCK, (int64_t)ctx->num_cus * BLOCKS_PER_CU);
    Arena a;
    auto plan = [&](Arena& ar) {
        if (!lds) {
            d.bits = ar.zero<uint32_t>(flags_direct_words(f));
            d.extra = ar.zero<uint32_t>(int64_t(1) << norm_key_bits(f.key_bits));
            d.repeats = ar.zero<uint32_t>(1);
        }
        d.part = ar.scratch<int64_t>(FLAGS_PART * d.nslot);
    };
    tqp_status st = with_workspace(ctx, ws, ws_bytes, s, plan, a);
    if (st != TQP_OK || !ws) return st;
    if (lds) {
        TQP_LAUNCH(ctx, s, "flags_fact_lds", k_flags_fact_lds<<<(unsigned)d.nslot, BLOCK, 0, s>>>(d, ctx->d_err));
    } else {
        if ((st = fill_zero(a.base, a.zsize, s, ctx)) != TQP_OK) return st;
        if (f.n_dim > 0)
            TQP_LAUNCH(ctx, s, "flags_dim",
                       k_flags_dim<<<grid_for(f.n_dim, BLOCK, (int64_t)ctx->num_cus * 8), BLOCK, 0, s>>>(d, ctx->d_err));
        TQP_LAUNCH(ctx, s, "flags_fact", k_flags_fact<<<(unsigned)d.nslot, BLOCK, 0, s>>>(d, ctx->d_err));
    }
    TQP_LAUNCH(ctx, s, "flags_finalize", k_flags_direct_final<<<1, FINAL_BLOCK, 0, s>>>(d));
    return TQP_OK;
}

tqp_status flags_direct_batch(tqp_ctx* ctx, const FlagsDirect* frags, int nfrag, const FlagsItem* dim_items,
                              int64_t ndim_items, const FlagsItem* fact_items, int64_t nfact_items, hipStream_t s) {
    if (ndim_items > 0)
        TQP_LAUNCH(ctx, s, "batch_flags_dim",
                   k_batch_flags_dim<<<(unsigned)ndim_items, BLOCK, 0, s>>>(frags, dim_items, ctx->d_err));
    if (nfact_items > 0)
        TQP_LAUNCH(ctx, s, "batch_flags_fact",
                   k_batch_flags_fact<<<(unsigned)nfact_items, BLOCK, 0, s>>>(frags, fact_items, ctx->d_err));
    if (nfrag > 0)
        TQP_LAUNCH(ctx, s, "batch_flags_final",
                   k_batch_flags_final<<<(unsigned)nfrag, FINAL_BLOCK, 0, s>>>(frags));
    return TQP_OK;
}

}  // namespace tqp
