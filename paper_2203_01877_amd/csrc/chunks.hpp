// Partitioning into chunk lists: (key, value) rows moved into 2^bits
// partitions by the top bits of their key, in one pass and with no count of
// the partitions beforehand.  Rows of one partition need not be contiguous:
// they lie in chunks of CHUNK rows, and every block fills chunks of its own,
// one open per partition, so that consecutive tiles of a block extend the
// same lines.  A tile draws the new chunks of all its partitions with one
// atomic on the pool.  Row order within a partition is not kept, so this
// serves consumers that do not depend on it (joins by table, aggregations),
// where a sort pass would need the partitions' counts first (a read of every
// key) and the tiles' offsets (a look-back per tile).
#pragma once
#include "chunkpool.hpp"
#include "dev.hpp"
#include "host.hpp"
#include "radix.hpp"

namespace tqp {

constexpr int CHUNK_GROUP = 4096 / CHUNK;      // chunks a wave takes at a time, one number per lane
constexpr int PART_BLOCK = 512;
constexpr int PART_WAVES = 4;          // waves per SIMD: two blocks per CU, at most 128 VGPRs
constexpr int PART_MAX_BITS = 8;
constexpr int PART_MAX = 1 << PART_MAX_BITS;
constexpr uint32_t PART_NONE = ~0u;    // the key of an item that takes no part (keys have at most 31 bits)
constexpr int PART_BLOCKS_PER_CU = 2;  // what the staged tile leaves room for

// Rows per thread: tiles of 8192 rows with a 4-byte value, 6144 with an
// 8-byte one (64 and 72 KB staged, two blocks per CU).
template <class V> struct PartItems { static constexpr int value = sizeof(V) <= 4 ? 16 : 12; };
template <class V> constexpr int part_tile() { return PART_BLOCK * PartItems<V>::value; }

// A chunk list.  KT: uint32_t, or uint16_t when the bits below the partition
// number fit it.
template <class KT, class V>
struct Chunks {
    KT* keys = nullptr;                // [nchunk][CHUNK] key bits below the partition number (KT = uint16_t), or whole keys
    V* vals = nullptr;                 // [nchunk][CHUNK]
    uint8_t* label = nullptr;          // [nchunk] partition of each chunk
    uint32_t* rows = nullptr;          // [nchunk] rows in each chunk
    uint32_t* list = nullptr;          // [nchunk] the chunks by partition (after chunks_list)
    uint32_t* first = nullptr;         // [partitions] first entry of each partition in the list
    uint32_t* dcount = nullptr;        // [partitions] chunks of each partition (zero on entry)
    uint32_t* cursor = nullptr;        // [partitions] chunks listed (zero on entry)
    uint64_t* pool = nullptr;          // [POOL_WORDS] rows and chunks claimed, rows past the capacity (zero on entry)
    uint32_t* open = nullptr;          // [nblocks][partitions] each block's open chunks, or null (part_reopen)
    int64_t nchunk = 0;                // chunks in the pool
    int64_t row_cap = 0;               // rows beyond this are counted but not kept
    int shift = 0;                     // partition = key >> shift
    int part_bits = 0;
    int nblocks = 0;                   // blocks that fill it
};

inline int part_blocks(const tqp_ctx* ctx, int64_t n, int tile) {
    return grid_for(n, tile, (int64_t)ctx->num_cus * PART_BLOCKS_PER_CU);
}

// Partition bits, at most max_bits, at which the chunks that nblocks blocks
// may leave part-filled hold no more rows than the input: a small input has
// few rows per block, and spreading them over more chunks costs scratch and
// lane-filling reads.
inline int part_bits_for(int64_t rows, int nblocks, int max_bits) {
    int bits = 4;
    while (bits < max_bits && ((int64_t)nblocks * CHUNK << (bits + 1)) <= rows) ++bits;
    return bits < max_bits ? bits : max_bits;
}

// row_cap rows from at most nblocks blocks.
template <class KT, class V>
void chunks_reserve(Arena& a, Chunks<KT, V>& c, int64_t row_cap, int nblocks, int key_bits, int part_bits) {
    const int parts = 1 << part_bits;
    c.row_cap = row_cap;
    c.nblocks = nblocks;
    c.part_bits = part_bits;
    c.shift = key_bits - part_bits;
    c.nchunk = pool_chunks(row_cap, nblocks, parts, part_tile<V>());
    c.dcount = a.zero<uint32_t>(parts);
    c.cursor = a.zero<uint32_t>(parts);
    c.pool = a.zero<uint64_t>(POOL_WORDS);
    c.keys = a.scratch<KT>(c.nchunk * CHUNK);
    c.vals = a.scratch<V>(c.nchunk * CHUNK);
    c.label = a.scratch<uint8_t>(c.nchunk);
    c.rows = a.scratch<uint32_t>(c.nchunk);
    c.list = a.scratch<uint32_t>(c.nchunk);
    c.first = a.scratch<uint32_t>(parts);
}

// ------------------------------------------------------------------ one tile
// A tile is the work of a block of PART_BLOCK threads, or of more threads with
// fewer items each.
template <class V, int BLOCK = PART_BLOCK>
struct PartSmem {
    static constexpr int TILE = PART_BLOCK * PartItems<V>::value, ITEMS = TILE / BLOCK;
    V vals[TILE];
    uint32_t keys[TILE];
    uint32_t cnt[PART_MAX];            // rows of the tile per partition
    uint32_t cur[PART_MAX];            // the block's open chunk per partition
    uint32_t at1[PART_MAX];            // address of staged row p: at1 + p before split, at2 + p from there on
    uint32_t at2[PART_MAX];
    uint16_t start[PART_MAX];          // first staged row of the partition
    uint16_t split[PART_MAX];
    uint16_t end[PART_MAX];            // staged rows from here on are not kept (beyond row_cap)
    uint16_t fill[PART_MAX];           // rows in the open chunk (CHUNK: none open)
    uint32_t scratch[BLOCK / WAVE];
    uint64_t claim;
    uint64_t over;                     // rows counted after the capacity was reached
    uint32_t full;                     // it was: the block claims nothing more
};

template <class KT, class V, int BLOCK>
__device__ __forceinline__ void part_init(PartSmem<V, BLOCK>& sm) {
    for (int d = threadIdx.x; d < PART_MAX; d += BLOCK) {
        sm.fill[d] = CHUNK;
        sm.cur[d] = 0;
    }
    if (threadIdx.x == 0) sm.over = sm.full = 0;
}

// Moves the block's tile (the items of each thread whose key is not PART_NONE)
// into the chunk list; false, to the whole block, once the list's capacity is
// reached (a later tile's rows are then only counted).  Called by the whole
// block.
template <class KT, class V, int BLOCK>
__device__ __forceinline__ bool part_tile_rows(const Chunks<KT, V>& out, int parts,
                                               const uint32_t (&key)[PartSmem<V, BLOCK>::ITEMS],
                                               const V (&val)[PartSmem<V, BLOCK>::ITEMS], PartSmem<V, BLOCK>& sm) {
    constexpr int ITEMS = PartSmem<V, BLOCK>::ITEMS;
    int tid = threadIdx.x, shift = out.shift;
    // opaque, so that what follows from them is not kept in registers from
    // one tile to the next (143 VGPRs: one block per CU instead of two)
    asm volatile("" : "+v"(tid));
    asm volatile("" : "+s"(shift));
    if (tid < PART_MAX) sm.cnt[tid] = 0;
    __syncthreads();                   // also: the previous tile's rows are written out
    if (sm.full) {
        uint32_t n = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) n += popc64(ballot(key[j] != PART_NONE));
        if (lane_id() == 0 && n) atomicAdd(reinterpret_cast<unsigned long long*>(&sm.over), (unsigned long long)n);
        return false;
    }
    uint32_t pos[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (key[j] != PART_NONE) pos[j] = atomicAdd(&sm.cnt[key[j] >> shift], 1u);
    __syncthreads();
    // partition starts in the tile and new chunks, in one scan (the tile's
    // rows in the low half, the chunks in the high half)
    uint32_t c = 0, need = 0, room = 0;
    if (tid < parts) {
        c = sm.cnt[tid];
        room = CHUNK - sm.fill[tid];
        need = chunks_needed(c, sm.fill[tid]);
    }
    uint32_t tot;
    const uint32_t excl = block_excl_sum<BLOCK>((need << 16) | c, sm.scratch, &tot);
    const uint32_t total = tot & 0xFFFFu;
    uint64_t claim = 0;                // in flight while the tile is staged
    if (tid == 0)
        claim = __hip_atomic_fetch_add(out.pool, pool_add(total, tot >> 16), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t s = excl & 0xFFFFu;
    if (tid < parts) sm.start[tid] = (uint16_t)s;
    __syncthreads();
    // stage in partition order
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (key[j] != PART_NONE) {
            const uint32_t p = sm.start[key[j] >> shift] + pos[j];
            sm.keys[p] = key[j];
            sm.vals[p] = val[j];
        }
    }
    if (tid == 0) sm.claim = claim;
    __syncthreads();
    const PoolClaim pc = pool_claim(sm.claim, total, tot >> 16, out.row_cap, out.nchunk);
    const int64_t keep = pc.keep;
    const uint32_t base = (uint32_t)(pc.chunk0 + (excl >> 16));
    if (tid == 0) sm.full = pc.full;
    uint32_t added = 0;                // chunks the partition takes
    uint32_t full = ~0u;               // its open chunk, now full
    if (tid < parts) {
        // rows of this partition that are kept: all, unless the tile crosses row_cap
        const uint32_t ck = s >= keep ? 0 : s + c > keep ? (uint32_t)keep - s : c;
        const uint32_t first = ck < room ? ck : room;
        sm.split[tid] = (uint16_t)(s + first);
        sm.end[tid] = (uint16_t)(s + ck);
        sm.at1[tid] = sm.cur[tid] * CHUNK + sm.fill[tid] - s;
        sm.at2[tid] = base * CHUNK - (s + first);
        uint32_t fill = sm.fill[tid] + first;
        if (first && fill == CHUNK) full = sm.cur[tid];
        if (ck > room) {
            added = (ck - room + CHUNK - 1) / CHUNK;
            sm.cur[tid] = base + added - 1;
            fill = ck - room - (added - 1) * CHUNK;
        }
        sm.fill[tid] = (uint16_t)fill;
    }
    __syncthreads();
    // every chunk but an open one is full
    if (full != ~0u) out.rows[full] = CHUNK;
    // every chunk claimed gets a label, so that the list holds each one; the
    // rows a tile drops at row_cap may leave some of them empty
    const uint32_t claimed = chunks_in_pool(base, need, out.nchunk);
    if (tid < parts && claimed) {
        atomic_add(&out.dcount[tid], claimed);
        for (uint32_t i = 0; i < claimed; ++i) {
            out.label[base + i] = (uint8_t)tid;
            if (i >= added) out.rows[base + i] = 0;
            else if (i + 1 < added || sm.fill[tid] == CHUNK) out.rows[base + i] = CHUNK;
        }
    }
    // consecutive staged rows of one partition go to consecutive addresses
#pragma unroll 4
    for (uint32_t p = tid; p < total; p += BLOCK) {
        const uint32_t k = sm.keys[p];
        const uint32_t d = k >> shift;
        if (p < sm.end[d]) {
            const uint32_t g = p + (p < sm.split[d] ? sm.at1[d] : sm.at2[d]);
            out.keys[g] = (KT)(sizeof(KT) == 2 ? k & ((1u << shift) - 1) : k);
            out.vals[g] = sm.vals[p];
        }
    }
    return !pc.full;
}

// Row counts of the chunks the block leaves part-filled, and where they are;
// the rows it counted past the capacity.  Called by the whole block.
template <class KT, class V, int BLOCK>
__device__ __forceinline__ void part_finish(const Chunks<KT, V>& out, int parts, PartSmem<V, BLOCK>& sm) {
    const int d = threadIdx.x;
    __syncthreads();
    if (d == 0 && sm.over) atomic_add(out.pool + 1, sm.over);
    if (d >= parts) return;
    if (sm.fill[d] < CHUNK) out.rows[sm.cur[d]] = sm.fill[d];
    if (out.open) out.open[(int64_t)blockIdx.x * parts + d] = sm.fill[d] < CHUNK ? sm.cur[d] : ~0u;
}

// In place of part_init, a later kernel's block: it goes on filling the chunks
// that the block of its number left open, so that the kernel adds no
// part-filled chunks.
template <class KT, class V, int BLOCK>
__device__ __forceinline__ void part_reopen(const Chunks<KT, V>& out, int parts, PartSmem<V, BLOCK>& sm) {
    for (int d = threadIdx.x; d < PART_MAX; d += BLOCK) {
        const uint32_t c = d < parts ? out.open[(int64_t)blockIdx.x * parts + d] : ~0u;
        sm.cur[d] = c != ~0u ? c : 0;
        sm.fill[d] = c != ~0u ? (uint16_t)out.rows[c] : CHUNK;
    }
    if (threadIdx.x == 0) sm.over = sm.full = 0;
}

// ------------------------------------------------------------------ the lists
// The chunks by partition: a counting sort of their labels, a block per 4096
// chunks.  (A list per partition, long enough for every chunk, would spare it,
// and cost 8 bytes of scratch per row.)
constexpr int LIST_BLOCK = 256, LIST_ITEMS = 16;
__global__ void k_chunks_list(const uint8_t* label, const uint64_t* pool, const uint32_t* dcount, uint32_t* cursor,
                              uint32_t* list, uint32_t* first, int parts, int64_t nchunk);

template <class KT, class V>
tqp_status chunks_list(tqp_ctx* ctx, hipStream_t s, const char* name, const Chunks<KT, V>& c) {
    TQP_LAUNCH(ctx, s, name,
               k_chunks_list<<<grid_for(c.nchunk, LIST_BLOCK * LIST_ITEMS, 0), LIST_BLOCK, 0, s>>>(
                   c.label, c.pool, c.dcount, c.cursor, c.list, c.first, 1 << c.part_bits, c.nchunk));
    return TQP_OK;
}

// ------------------------------------------------------------------ columns
// The wave's number, known to the compiler to be the same in every lane: what
// depends on it alone (chunk numbers, the start of a wave's rows) stays in
// scalar registers, and rows are read at a scalar base plus the lane.
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE); }

// Items of a wave: rows [base, base + ITEMS * 64) of the source, those past
// its end, those the source leaves out and those whose key lies outside
// key_mask marked PART_NONE.
template <class Src, class V, int ITEMS>
__device__ __forceinline__ void part_load(const Src& src, int64_t n, int64_t base, uint32_t (&key)[ITEMS],
                                          V (&val)[ITEMS], uint32_t key_mask, uint32_t& bad, uint32_t& bad_key) {
    int l = lane_id();
    asm volatile("" : "+v"(l));        // opaque, as in part_tile_rows
    auto row = [&](int j, int64_t i, bool in) {
        bool ok;
        if constexpr (SrcChecks<Src>::value) ok = src.load(i, key[j], val[j], bad);
        else ok = src.load(i, key[j], val[j]);
        ok = ok && in;
        const bool wide = (key[j] & ~key_mask) != 0;
        bad_key |= (uint32_t)(ok & wide);
        key[j] = ok & !wide ? key[j] : PART_NONE;
    };
    if (base + ITEMS * WAVE <= n) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) row(j, base + (j * WAVE + l), true);
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {              // clamped index: no branch between the loads
            const int64_t i = base + j * WAVE + l;
            row(j, i < n ? i : n - 1, i < n);
        }
    }
}

// Partition of a source's rows (radix.hpp's sources).  Rows whose key lies
// outside key_mask are left out and flagged.  Bound by HBM and by the staging
// of a tile between two barriers: two blocks of 8192 rows per CU hide more of
// each other's than four of 4096 (60M x 15M join in all 1422 and 1590 us), and
// written without the non-temporal hint the lines of a partition that
// consecutive tiles extend meet in L2 (1422 and 1573 us).  60M filtered fact
// rows (16 bytes read, 8 written) take 434 us, where the histogram and first
// pass of the sort took 606.
template <class KT, class V, class Src, int Tag = 0>
__global__ void __launch_bounds__(PART_BLOCK, PART_WAVES)
k_part(Src src, Chunks<KT, V> out, int parts, uint32_t key_mask, uint32_t* flags) {
    constexpr int ITEMS = PartItems<V>::value, TILE = PART_BLOCK * ITEMS;
    __shared__ PartSmem<V> sm;
    const int tid = threadIdx.x, w = wave_index(), l = lane_id();
    part_init<KT, V, PART_BLOCK>(sm);
    const int64_t n = src.size();
    const int64_t ntiles = (n + TILE - 1) / TILE;
    uint32_t bad = 0, bad_key = 0;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        uint32_t key[ITEMS];
        V val[ITEMS];
        part_load(src, n, tile * TILE + (int64_t)w * ITEMS * WAVE, key, val, key_mask, bad, bad_key);
        part_tile_rows<KT, V, PART_BLOCK>(out, parts, key, val, sm);
    }
    part_finish<KT, V, PART_BLOCK>(out, parts, sm);
    if (__any(bad_key != 0) && l == 0) set_flag(flags, FLAG_KEY_RANGE);
    if (__any(bad != 0) && l == 0) set_flag(flags, FLAG_VALUE_RANGE);
}

template <class KT, class V, int Tag = 0, class Src>
tqp_status part_launch(tqp_ctx* ctx, hipStream_t s, const char* name, const Src& src, int64_t n_upper,
                       const Chunks<KT, V>& out, uint32_t key_mask, const char* list_name) {
    if (n_upper > 0)
        TQP_LAUNCH(ctx, s, name,
                   (k_part<KT, V, Src, Tag><<<(unsigned)out.nblocks, PART_BLOCK, 0, s>>>(src, out, 1 << out.part_bits,
                                                                                       key_mask, ctx->d_err)));
    return chunks_list(ctx, s, list_name, out);
}

}  // namespace tqp
