"""The general fragment's pairs by a key table: tiles' edges, keys on several dim rows (short lists, and lists that
a kernel of their own writes), a join larger than its capacity, keys outside the width."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

AGGS = [(1, [(0, 1), (0, 4), (3, 0)]), (0, []), (2, [(0, 1)]), (3, [(0, 4)])]     # SUM(v * w), COUNT, MIN(v), MAX(w)


def _run(hip, ctx, fact, dim, key_bits, join_cap=None, gcap=12):
    import torch
    dev = lambda cs: [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cs]
    ctx.set_profiling(True)
    out = hip.fragment_run(ctx, dev(fact), dev(dim), [(0, 1), (1, 500), (8, 0)], [(0, 1), (1, 3), (13, 0)], 0, 0,
                           [(2, 2), (4, 2)], AGGS, key_bits=key_bits, gcap=gcap, join_cap=join_cap)
    assert "fragment_pairs" in [n for n, _ in ctx.profile_read()]
    ctx.set_profiling(False)
    return out


def _tables(n, m, hi, keys, seed):
    """fact (key, v, flag); dim (key, w in [0, 3)); v < 500 and w != 3 are the predicates."""
    r = np.random.default_rng(seed)
    fact = [r.integers(0, hi, n).astype(np.int32), r.integers(-1000, 1000, n).astype(np.int32),
            r.integers(0, 4, n).astype(np.int8)]
    pk = r.permutation(hi)[:m] if keys == "unique" else np.arange(m) // 2 if keys == "pairs" else np.arange(m)
    if keys == "hot":
        pk = pk.copy()
        pk[: m // 2] = 3                             # 3 on half the dim rows, 5 on 65 and 7 on 64 of them
        pk[m // 2: m // 2 + 65], pk[m // 2 + 65: m // 2 + 129] = 5, 7
        fact[0][:] = 8 + fact[0] % (hi - 8)
        fact[0][r.permutation(n)[:300]] = np.tile([3, 5, 7], 100)
    return fact, [pk.astype(np.int32), r.integers(0, 3, m).astype(np.int32)]


def _want(fact, dim):
    # the dim columns follow the fact's: column 4 is w
    return oracle.fragment_general(fact, dim, [(0, 1), (1, 500), (8, 0)], [(0, 1), (1, 3), (13, 0)], 0, 0,
                                   [(2, 2), (4, 2)], AGGS, topk=0, gcap=1 << 10)


@pytest.mark.parametrize("n,m,key_bits", [(1, 1, 1), (16_383, 300, 9), (16_385, 9_000, 15), (1_000_003, 300_000, 20)])
@pytest.mark.parametrize("keys", ["unique", "pairs", "hot"])
def test_pair_table(hip, n, m, key_bits, keys):
    if keys != "unique" and n < 1000:
        pytest.skip("one row")
    ctx = hip.Context(0)
    fact, dim = _tables(n, m, 1 << key_bits if n > 1 else 2, keys, n)
    want = _want(fact, dim)
    for _ in range(2):
        got = _run(hip, ctx, fact, dim, key_bits, join_cap=max(1, want["join_rows"]))
        g = int(got["d_ngroups"].item())
        assert ctx.errors() == 0 and g == want["groups"] and int(got["d_join"].item()) == want["join_rows"]
        assert np.array_equal(got["key"][:g].cpu().numpy(), want["key"])
        for a, b in zip(got["vals"], want["vals"]):
            assert np.array_equal(a[:g].cpu().numpy().view(np.int64), np.asarray(b).view(np.int64))


@pytest.mark.parametrize("keys", ["unique", "hot"])
@pytest.mark.parametrize("less", [1, 5_000])
def test_pair_table_capacity(hip, keys, less):
    """A capacity below the join's size: the true size, the flag, and exactly the capacity's rows counted."""
    ctx = hip.Context(0)
    fact, dim = _tables(100_000, 20_000, 1 << 15, keys, 5)
    rows = _want(fact, dim)["join_rows"]
    got = _run(hip, ctx, fact, dim, 15, join_cap=rows - less)
    assert ctx.errors() == hip.DEVERR_CAPACITY and int(got["d_join"].item()) == rows
    assert int(got["vals"][1][: int(got["d_ngroups"].item())].sum()) == rows - less


@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("bad", [-3, 1 << 15])
def test_pair_table_key_range(hip, side, bad):
    """A key outside the width is flagged when the row passes its side's predicate, and only then."""
    ctx = hip.Context(0)
    fact, dim = _tables(50_000, 9_000, 1 << 15, "unique", 6)
    t, col = (fact, 1) if side == 0 else (dim, 1)
    for kept in (True, False):
        t[0][17], t[col][17] = bad, (0 if kept else 900 if side == 0 else 3)
        _run(hip, ctx, fact, dim, 15, join_cap=50_000)
        assert ctx.errors() == (hip.DEVERR_KEY_RANGE if kept else 0)
