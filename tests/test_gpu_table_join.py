"""The custkey and keyed general fragments with their join by a key table, against the oracle, at the edges
of its rule and of its tiles: key domains from one key to the last without and the first with a fact
partition, group keys from one partition to 21 bits, tile remainders, keys with several dim rows (lists
shorter and longer than a tile), a dim side sorted by key, empty sides, keys and group keys outside their
width, and a join capacity below the join's size.  Every value is an integer and exact."""
import dataclasses

import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu


def _case(n, m, cust, seed=5):
    return datagen.config2(seed=seed, n=n, m=m, cust_hi=cust)


def _run(hip, ctx, fr, key_bits, cust_bits, rbits=32, cap=None, sorted_=False, gcap=None):
    """The fragment run once by the table (asserted by the names of its launches)."""
    mid = fr.mid
    if sorted_:
        o = np.argsort(mid["pk"], kind="stable")
        mid = {k: v[o] for k, v in mid.items()}
    r = hip.CustFragmentRunner(ctx, hip.to_device({k: fr.fact[k] for k in ("fk", "date", "price", "disc")}),
                               hip.to_device(mid), fr.D, fr.k, key_bits=key_bits, cust_bits=cust_bits,
                               gcap=gcap or max(1, min(max(len(fr.fact["fk"]), cap or 0), fr.cust_hi)),
                               join_cap=cap, revenue_bits=rbits, mid_sorted=sorted_)
    ctx.set_profiling(True)
    r.run()
    names = [n for n, _ in ctx.profile_read()]
    ctx.set_profiling(False)
    assert "probe" in names and ("fact_part" in names) == (key_bits > 20)
    return r


def _same(got, want):
    assert got["join_rows"] == want["join_rows"] and got["groups"] == want["groups"]
    for k in ("key", "sum", "cnt", "top_key", "top_sum", "top_cnt"):
        assert np.array_equal(got[k], want[k])


def _bits(fr):
    return datagen.bits_for(max(int(fr.fact["fk"].max(initial=0)), int(fr.mid["pk"].max(initial=0))) + 1)


@pytest.mark.parametrize("rbits", [32, 64])
@pytest.mark.parametrize("n,m,cust,key_bits", [
    (60_000, 1, 1, 1),                       # one key
    (8_192 * 9 - 1, 15_000, 1_500, 14),      # tiles of 4-byte values less one row
    (6_144 * 9 + 1, 15_000, 1_500, 14),      # tiles of 8-byte values and one row
    (300_000, 90_000, 70_000, 20),           # the last key domain probed without a fact partition
    (3_000_000, 800_000, 70_000, 21),        # the first with one
])
@pytest.mark.parametrize("sorted_", [False, True])
def test_table_edges(hip, n, m, cust, key_bits, rbits, sorted_):
    ctx = hip.Context(0)
    fr = _case(n, m, cust)
    want = oracle.fragment_cust(fr.fact, fr.mid, fr.D, fr.k, gcap=min(n, cust))
    cb = max(1, int(cust - 1).bit_length())
    got = _run(hip, ctx, fr, max(key_bits, _bits(fr)), cb, rbits, sorted_=sorted_)
    _same(got.result(), want)
    got.run()
    _same(got.result(), want)
    assert ctx.errors() == 0


@pytest.mark.parametrize("rbits", [32, 64])
@pytest.mark.parametrize("shape", ["pairs", "hot", "few"])
@pytest.mark.parametrize("key_bits", [18, 21])
def test_table_lists(hip, shape, key_bits, rbits):
    """Keys with several dim rows: every key on two, one key on 20,000 (its list longer than a tile), and
    dim rows on three keys only."""
    ctx = hip.Context(0)
    n, m = (400_000, 150_000) if key_bits == 18 else (3_000_000, 800_000)
    fr = _case(n, m, 9_000, seed=6)
    pk, fk = fr.mid["pk"].copy(), fr.fact["fk"].copy()
    if shape == "pairs":
        pk //= 2
    elif shape == "hot":
        pk[:20_000] = 77
    else:
        pk = (pk % 3).astype(np.int32)
        fk[400:] = 3 + fk[400:] % (m - 3)    # 400 rows may meet them, with a third of the dim rows each
        fk[:400] %= 5
    fr = dataclasses.replace(fr, mid=dict(fr.mid, pk=pk), fact=dict(fr.fact, fk=fk))
    want = oracle.fragment_cust(fr.fact, fr.mid, fr.D, fr.k, gcap=fr.cust_hi)
    cap = want["join_rows"]
    got = _run(hip, ctx, fr, max(key_bits, _bits(fr)), 14, rbits, cap=cap, gcap=fr.cust_hi)
    _same(got.result(), want)
    assert ctx.errors() == 0


@pytest.mark.parametrize("key_bits,n,cap", [(18, 300_000, 100_001), (21, 4_000_000, 1_500_001)])
def test_table_capacity(hip, key_bits, n, cap):
    """A capacity below the join's size: the true size, the flag, and exactly the capacity's rows counted."""
    ctx = hip.Context(0)
    fr = _case(n, n // 4, 5_000)
    want = oracle.fragment_cust(fr.fact, fr.mid, fr.D, fr.k, gcap=fr.cust_hi)
    assert want["join_rows"] > cap
    for _ in range(2):
        got = _run(hip, ctx, fr, key_bits, 13, 64, cap=cap, gcap=5_000).result()
        assert ctx.errors() == hip.DEVERR_CAPACITY
        assert got["join_rows"] == want["join_rows"] and int(got["cnt"].sum()) == cap


@pytest.mark.parametrize("side", ["fact", "mid"])
@pytest.mark.parametrize("bad", [-3, 1 << 21])
@pytest.mark.parametrize("key_bits", [19, 21])
def test_table_key_range(hip, side, bad, key_bits):
    """A key outside the declared width is flagged (on the fact side only when the row passes the filter)."""
    ctx = hip.Context(0)
    fr = _case(*((300_000, 100_000) if key_bits == 19 else (3_000_000, 800_000)), 5_000)
    t, col = (fr.fact, "fk") if side == "fact" else (fr.mid, "pk")
    key = t[col].copy()
    key[int(np.flatnonzero(fr.fact["date"] < fr.D)[5]) if side == "fact" else 17] = bad
    new = dataclasses.replace(fr, **{side: dict(t, **{col: key})})
    _run(hip, ctx, new, key_bits, 13)
    assert ctx.errors() == hip.DEVERR_KEY_RANGE
    if side == "fact":
        key = t[col].copy()
        key[int(np.flatnonzero(fr.fact["date"] >= fr.D)[5])] = bad
        new = dataclasses.replace(fr, fact=dict(t, fk=key))
        got = _run(hip, ctx, new, key_bits, 13)
        assert ctx.errors() == 0
        _same(got.result(), oracle.fragment_cust(fr.fact, fr.mid, fr.D, fr.k, gcap=fr.cust_hi))


def test_table_group_range(hip):
    """A custkey outside its width is flagged when its row joins, and only then."""
    ctx = hip.Context(0)
    fr = _case(300_000, 100_000, 5_000)
    hit = np.isin(fr.mid["pk"], fr.fact["fk"][fr.fact["date"] < fr.D])
    for joins in (True, False):
        ck = fr.mid["custkey"].copy()
        ck[np.flatnonzero(hit == joins)[3]] = 1 << 13
        _run(hip, ctx, dataclasses.replace(fr, mid=dict(fr.mid, custkey=ck)), 18, 13)
        assert ctx.errors() == (hip.DEVERR_KEY_RANGE if joins else 0)


@pytest.mark.parametrize("vbits", [0, 32])
@pytest.mark.parametrize("op", ["SUM", "MIN", "MAX", "AVG"])
def test_table_general(hip, op, vbits):
    """The keyed general fragment: predicates on both sides, signed values, every valued aggregate."""
    ctx = hip.Context(0)
    ctx.set_profiling(True)
    X, agg = oracle, {"SUM": 1, "MIN": 2, "MAX": 3, "AVG": 4}[op]
    fr = _case(400_000, 100_000, 70_000, seed=9)
    price = (fr.fact["price"] - 5_000_000).astype(np.int64)
    fact = [fr.fact["fk"], fr.fact["date"], price]
    dim = [fr.mid["pk"], fr.mid["custkey"]]
    fp = [(0, 1), (1, 2000), (8, 0)]                     # date < 2000
    dp = [(0, 1), (1, 3), (6, 0), (1, 0), (13, 0)]       # custkey % 3 != 0
    aggs = [(agg, [(0, 2), (1, 7), (3, 0)]), (0, [])]    # over price - 7, and COUNT
    topk = 0 if op == "AVG" else 20
    want = X.fragment_general(fact, dim, fp, dp, 0, 0, [(4, 17)], aggs, topk=topk, gcap=1 << 20)
    import torch
    dev = lambda cs: [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cs]
    out = hip.fragment_run(ctx, dev(fact), dev(dim), fp, dp, 0, 0, [(4, 17)], aggs, topk=topk, key_bits=18,
                           gcap=max(1, want["groups"]), value_bits=vbits)
    assert int(out["d_ngroups"].item()) == want["groups"] and int(out["d_join"].item()) == want["join_rows"]
    assert np.array_equal(out["key"].cpu().numpy(), want["key"])
    for a, b in zip(out["vals"], want["vals"]):
        assert np.array_equal(a.cpu().numpy().view(np.int64), np.asarray(b).view(np.int64))
    assert "fragment_probe" in [n for n, _ in ctx.profile_read()]
    if topk:
        assert np.array_equal(out["top_key"].cpu().numpy(), want["top_key"])
        assert np.array_equal(out["top_val"].cpu().numpy(), want["top_val"])
    assert ctx.errors() == 0
