"""The claim arithmetic of the chunk lists (csrc/chunkpool.hpp, compiled here for the host), walked through joins
far larger than their capacity: no chunk is given out twice, the lists hold no more chunks than the pool, exactly
the capacity's rows are kept, and every row is counted.  A block that went on claiming for the rows it drops would
wrap the chunk number after about 2^31 of them; the same walk without the stop shows that."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2203_01877_amd", "csrc")

WALK = r"""
#define __host__
#define __device__
#include "chunkpool.hpp"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace tqp;

// argv: rows, row_cap, parts, nblocks, tile, stop
int main(int, char** a) {
    const int64_t rows = atoll(a[1]), row_cap = atoll(a[2]);
    const int parts = atoi(a[3]), nblocks = atoi(a[4]), tile = atoi(a[5]), stop = atoi(a[6]);
    const int64_t nchunk = pool_chunks(row_cap, nblocks, parts, tile);
    std::vector<uint8_t> labelled(nchunk, 0);
    std::vector<int64_t> in_chunk(nchunk, 0);
    std::vector<uint32_t> fill((size_t)nblocks * parts, CHUNK), cur((size_t)nblocks * parts, 0);
    std::vector<char> full(nblocks, 0);
    uint64_t pool[POOL_WORDS] = {0, 0}, rnd = 88172645463325252ull;
    int64_t dcount = 0, kept = 0, twice = 0;
    auto next = [&] { rnd ^= rnd << 13; rnd ^= rnd >> 7; rnd ^= rnd << 17; return rnd; };
    std::vector<uint32_t> cnt(parts), need(parts), excl(parts), start(parts);
    for (int64_t left = rows; left > 0;) {
        const int b = (int)(next() % nblocks);
        uint32_t total = left < tile ? (uint32_t)left : next() % 8 ? (uint32_t)tile : (uint32_t)(next() % tile + 1);
        left -= total;
        if (full[b] && stop) { pool[1] += total; continue; }
        uint32_t chunks = 0, s = 0;
        for (int d = 0; d < parts; ++d) {          // an even share each, the rest to one of them
            cnt[d] = total / parts;
        }
        cnt[next() % parts] += total % parts;
        for (int d = 0; d < parts; ++d) {
            start[d] = s;
            s += cnt[d];
            need[d] = chunks_needed(cnt[d], fill[(size_t)b * parts + d]);
            excl[d] = chunks;
            chunks += need[d];
        }
        const uint64_t word = pool[0];
        pool[0] += pool_add(total, chunks);
        const PoolClaim c = pool_claim(word, total, chunks, row_cap, nchunk);
        full[b] = c.full;
        for (int d = 0; d < parts; ++d) {
            uint32_t &f = fill[(size_t)b * parts + d], &o = cur[(size_t)b * parts + d];
            const uint32_t base = (uint32_t)(c.chunk0 + excl[d]);
            const uint32_t in = chunks_in_pool(base, need[d], nchunk);
            dcount += in;
            for (uint32_t i = 0; i < in; ++i) {
                twice += labelled[base + i];
                labelled[base + i] = 1;
            }
            int64_t k = c.keep - start[d];
            k = k < 0 ? 0 : k > cnt[d] ? cnt[d] : k;
            kept += k;
            while (k > 0) {                        // the open chunk, then the claimed ones
                const int64_t room = CHUNK - f, put = k < room ? k : room;
                if (room) in_chunk.at(o) += put;
                f += (uint32_t)put;
                k -= put;
                if (k > 0) {
                    o = f == CHUNK && in_chunk.at(o) == CHUNK && o >= base && o < base + need[d] ? o + 1 : base;
                    f = 0;
                }
            }
        }
    }
    for (int64_t n : in_chunk) if (n > CHUNK) return 2;
    if (pool_rows(pool[0], pool[1]) != rows) { printf("rows %lld\n", (long long)pool_rows(pool[0], pool[1])); return 3; }
    if (kept != (rows < row_cap ? rows : row_cap)) { printf("kept %lld\n", (long long)kept); return 4; }
    if (twice || dcount > nchunk) { printf("twice %lld dcount %lld of %lld\n", (long long)twice, (long long)dcount, (long long)nchunk); return 5; }
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("pool")
    (d / "walk.cpp").write_text(WALK)
    exe = str(d / "walk")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, "-o", exe, str(d / "walk.cpp")], check=True)

    def run(*args):
        return subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=300)
    return run


@pytest.mark.parametrize("rows,cap,parts,nblocks,tile", [
    (10 ** 10, 4_000_000, 16, 512, 8192),          # 1e10 pairs of keys frequent on both sides
    (10 ** 10, 4_000_000, 128, 512, 8192),
    (10 ** 10, 60_000_000, 256, 512, 6144),
    (10 ** 10, 0, 16, 512, 8192),                  # no room at all
    (12 * 10 ** 11, 1_000_000, 16, 256, 8192),       # more rows than the first word's 40 bits
    (4_000_000, 4_000_000, 16, 512, 8192),         # exactly the capacity
    (3_999_999, 4_000_000, 256, 512, 6144),
    (1, 1, 1, 1, 8192),
])
def test_claims(walk, rows, cap, parts, nblocks, tile):
    r = walk(rows, cap, parts, nblocks, tile, 1)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("cap,parts", [(4_000_000, 16), (60_000_000, 256)])
def test_claims_past_the_capacity_wrap(walk, cap, parts):
    assert walk(3 * 10 ** 9, cap, parts, 512, 8192, 0).returncode == 5
