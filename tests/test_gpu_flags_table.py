"""Flags fragments over a small key domain (no sorts: a table over the keys) against the oracle, at the
edges of its rule: the largest domain and dim side a fact block counts itself, the first beyond them, the
largest domain the table takes and the first left to the sorts.  Integers and averages are exact."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu


def _same(got, want):
    assert got["join_rows"] == want["join_rows"]
    for k in ("key", "sum", "cnt"):
        assert np.array_equal(got[k], want[k])
    assert np.array_equal(got["avg"].view(np.int64), want["avg"].view(np.int64))


@pytest.mark.parametrize("n,m,fk_hi,key_bits,dup", [
    (1, 1, 1, 1, False),                        # one row, one key
    (511, 4096, 4096, 12, False),               # counted in LDS: largest domain and dim side
    (513, 4097, 4097, 13, False),               # one more of each: the table
    (5000, 4096, 300, 12, True),                # LDS, keys that repeat
    (70_001, 9_001, 700, 13, True),             # table, keys that repeat
    (200_003, 3_000, 3_000, 18, False),         # 2^18 keys: the part of the rule without dim rows
    (200_003, 3_000, 3_000, 19, False),         # 2^19: the sorts
    (100_000, 70_000, 70_000, 19, False),       # 2^19 keys of 70k dim rows: the table
    (30_000, 2_000, 2_000, 0, False),           # undeclared width: the sorts
])
def test_flags_table_edges(hip, n, m, fk_hi, key_bits, dup):
    ctx = hip.Context(0)
    fr = datagen.random_flags_fragment(900 + n % 97, n, m, fk_hi, 2000, 1, dup_dim=dup)
    row0 = min(n - 1, 3)                        # columns from an odd row on
    fact, dim = hip.to_device(fr.fact), hip.to_device(fr.dim)
    want = oracle.fragment_flags({k: v[row0:] for k, v in fr.fact.items()}, fr.dim, fr.D, fr.c)
    r = hip.FlagsFragmentRunner(ctx, fact, dim, fr.D, fr.c, key_bits, row0=row0)
    b = hip.BatchRunner(ctx, [{"fact": fact, "dim": dim, "D": fr.D, "c": fr.c, "key_bits": key_bits, "row0": row0}])
    for _ in range(2):
        r.run()
        _same(r.result(), want)
        b.run()
        _same(b.results()[0], want)
    assert ctx.errors() == 0
    b.close()


@pytest.mark.parametrize("key_bits", [11, 14, 20])
@pytest.mark.parametrize("side", ["fact", "dim"])
def test_flags_table_key_range(hip, key_bits, side):
    """A key outside the declared width is flagged when its row passes the predicate, and only then."""
    ctx = hip.Context(0)
    fr = datagen.random_flags_fragment(77, 40_000, 1500, 1500, 2000, 1)
    table, col, pred = (fr.fact, "fk", fr.fact["date"] < 2000) if side == "fact" else (fr.dim, "pk", fr.dim["seg"] == 1)
    for keep, bad in ((False, -5), (True, 1 << key_bits), (True, -5)):
        key = table[col].copy()
        key[np.flatnonzero(pred == keep)[7]] = bad
        t = {**table, col: key}
        fact, dim = (t, fr.dim) if side == "fact" else (fr.fact, t)
        r = hip.FlagsFragmentRunner(ctx, hip.to_device(fact), hip.to_device(dim), fr.D, fr.c, key_bits)
        r.run()
        assert ctx.errors() == (hip.DEVERR_KEY_RANGE if keep else 0)
        if not keep:
            _same(r.result(), oracle.fragment_flags(fr.fact, fr.dim, fr.D, fr.c))


@pytest.mark.parametrize("mixed", [False, True])
def test_flags_table_batch(hip, mixed):
    """A batch whose fragments all take the table, and one with a fragment that does not; captured and
    replayed with the program's own work in between."""
    import torch
    ctx = hip.Context(0)
    frags, wants = [], []
    for i, (n, m) in enumerate([(16_384, 400), (16_385, 1), (0, 50), (100_000, 2_500), (3, 3)]):
        fr = datagen.random_flags_fragment(50 + i, n, m, m, 300 * i, i % 5)
        frags.append({"fact": hip.to_device(fr.fact), "dim": hip.to_device(fr.dim), "D": fr.D, "c": fr.c,
                      "key_bits": 0 if mixed and i == 3 else 13})
        wants.append(oracle.fragment_flags(fr.fact, fr.dim, fr.D, fr.c))
    b = hip.BatchRunner(ctx, frags)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b.capture(s)
        for _ in range(3):
            for v in b.out.values():
                v.fill_(-1)
            b.replay(s)
            s.synchronize()
            for got, want in zip(b.results(), wants):
                _same(got, want)
    assert ctx.errors() == 0
    b.close()
