// The arithmetic of a chunk list's pool (chunks.hpp): what a tile claims, what
// of it is kept, and when a block stops claiming.  Plain integers, the same on
// the host, where a test walks it through more rows than a GPU run would.
#pragma once
#include <cstdint>

namespace tqp {

// Rows per chunk.  Every block leaves a chunk of each partition part-filled:
// at 60M rows in 143 partitions by 512 blocks the lists are 75% full with 256
// rows per chunk and 86% with 128, and the probe over them takes 483 and
// 444 us.
constexpr int CHUNK = 128;

// The pool's first word counts what tiles have claimed: rows in the low 40
// bits, chunks above them.  Neither half can run over: a block that meets the
// capacity claims nothing more (PoolClaim::full), so that at most one tile per
// block is claimed beyond it; its later rows are counted in the second word.
constexpr int POOL_ROW_BITS = 40;
constexpr uint64_t POOL_ROW_MASK = (uint64_t(1) << POOL_ROW_BITS) - 1;
constexpr int POOL_WORDS = 2;

__host__ __device__ inline uint64_t pool_add(uint32_t rows, uint32_t chunks) {
    return ((uint64_t)chunks << POOL_ROW_BITS) | rows;
}
// Rows counted by the two words.
__host__ __device__ inline int64_t pool_rows(uint64_t claimed, uint64_t over) {
    return (int64_t)((claimed & POOL_ROW_MASK) + over);
}
// Chunks needed for row_cap rows from nblocks blocks: every block may leave
// one chunk of each partition part-filled, and the tile that crosses row_cap
// claims chunks for rows it drops.
inline int64_t pool_chunks(int64_t row_cap, int nblocks, int parts, int tile) {
    return row_cap / CHUNK + (int64_t)nblocks * parts + tile / CHUNK + 1;
}

// Chunks that c more rows of a partition take when its open chunk holds fill.
__host__ __device__ inline uint32_t chunks_needed(uint32_t c, uint32_t fill) {
    const uint32_t room = CHUNK - fill;
    return c > room ? (c - room + CHUNK - 1) / CHUNK : 0;
}

// A tile's claim of `rows` rows and `chunks` chunks, which found `word` in the
// pool: its first chunk, how many of its rows are kept, and whether the
// capacity is reached, after which the block only counts its rows.
struct PoolClaim {
    int64_t chunk0, keep;
    bool full;
};
__host__ __device__ inline PoolClaim pool_claim(uint64_t word, uint32_t rows, uint32_t chunks, int64_t row_cap,
                                                int64_t nchunk) {
    const int64_t row0 = (int64_t)(word & POOL_ROW_MASK);
    PoolClaim c;
    c.chunk0 = (int64_t)(word >> POOL_ROW_BITS);
    c.keep = row_cap - row0;
    if (c.keep > rows) c.keep = rows;
    if (c.keep < 0 || c.chunk0 + chunks > nchunk) c.keep = 0;
    c.full = row0 + rows >= row_cap;
    return c;
}
// Of `need` chunks claimed from `base` on, those that lie in the pool (they
// get a label, so that the list holds each one).
__host__ __device__ inline uint32_t chunks_in_pool(uint32_t base, uint32_t need, int64_t nchunk) {
    return base < nchunk ? (need < nchunk - base ? need : (uint32_t)(nchunk - base)) : 0;
}

}  // namespace tqp
