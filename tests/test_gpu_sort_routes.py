"""The sorts and joins that the fragments take without a key table, which undeclared or wide key widths (the
bindings' default among them) lead to: flags with and without the dim side's side stream, batches under every
configuration, custkey and general fragments at 8-bit digits, and the server.  The route is asserted by the names of
its launches; every value is exact."""
import dataclasses

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


def _names(ctx, run):
    ctx.set_profiling(True)
    run()
    names = {n for n, _ in ctx.profile_read()}
    ctx.set_profiling(False)
    return names


@pytest.mark.parametrize("key_bits", [0, 27])
@pytest.mark.parametrize("n,m,dup", [
    (1, 1, False), (5_000, 300, True), (90_001, 9_001, False),
    (120_000, 32_767, True), (120_000, 32_768, False),         # the dim sort on the side stream from here on
    (300_007, 70_001, True),
])
def test_flags(hip, n, m, dup, key_bits):
    ctx = hip.Context(0)
    fr = datagen.random_flags_fragment(700 + m % 83, n, m, m, 2000, 1, dup_dim=dup)
    row0 = min(n - 1, 5)
    want = oracle.fragment_flags({k: v[row0:] for k, v in fr.fact.items()}, fr.dim, fr.D, fr.c)
    r = hip.FlagsFragmentRunner(ctx, hip.to_device(fr.fact), hip.to_device(fr.dim), fr.D, fr.c, key_bits, row0=row0)
    assert "join_flags_agg" in _names(ctx, r.run)
    for _ in range(3):
        r.run()
        _same(r.result(), want)
    assert ctx.errors() == 0


@pytest.fixture(scope="module")
def wide_batch(hip):
    frags, wants = [], []
    for i, (n, m) in enumerate([(2_047, 40), (2_049, 1), (0, 50), (4_097, 4_096), (100_000, 2_500), (3, 3),
                                (250_001, 30_000), (60_000, 60_000)]):
        fr = datagen.random_flags_fragment(60 + i, n, m, m, 300 * i, i % 5, dup_dim=i % 3 == 0)
        frags.append({"fact": hip.to_device(fr.fact), "dim": hip.to_device(fr.dim), "D": fr.D, "c": fr.c,
                      "key_bits": 0 if i % 2 else 17})
        wants.append(oracle.fragment_flags(fr.fact, fr.dim, fr.D, fr.c))
    return frags, wants


@pytest.mark.parametrize("config", [0, 1, 2, 3])
def test_batch_configs(hip, wide_batch, config):
    frags, wants = wide_batch
    ctx = hip.Context(0)
    b = hip.BatchRunner(ctx, frags)
    b.set_config(config)
    names = _names(ctx, b.run)
    assert "batch_join" in names and "batch_flags_fact" not in names
    for _ in range(2):
        for got, want in zip(b.results(), wants):
            _same(got, want)
        b.run()
    assert ctx.errors() == 0
    b.close()


def test_batch_autotune_and_replay(hip, wide_batch):
    import torch
    frags, wants = wide_batch
    ctx = hip.Context(0)
    b = hip.BatchRunner(ctx, frags)
    times = b.autotune(reps=3)
    assert times[b.config()[2]] == min(times.values()) and len(set(times.values())) > 1
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


@pytest.mark.parametrize("rbits", [32, 64])
@pytest.mark.parametrize("mid", ["unique", "twice", "sorted"])
@pytest.mark.parametrize("n,m,key_bits,cust,cust_bits", [
    (8_193, 1_000, 0, 500, 9), (300_001, 80_003, 0, 70_000, 17), (500_000, 120_000, 28, 9_000, 0),
    (700_003, 200_001, 24, 70_000, 22),
])
def test_custkey(hip, n, m, key_bits, cust, cust_bits, mid, rbits):
    """Undeclared keys, a domain beyond the table's, group keys beyond its partitions."""
    ctx = hip.Context(0)
    fr = datagen.config2(seed=m, n=n, m=m, cust_hi=cust)
    t = dict(fr.mid, pk=fr.mid["pk"] // 2) if mid == "twice" else fr.mid
    if mid == "sorted":
        o = np.argsort(t["pk"], kind="stable")
        t = {k: v[o] for k, v in t.items()}
    fr = dataclasses.replace(fr, mid=t)
    want = oracle.fragment_cust(fr.fact, fr.mid, fr.D, fr.k, gcap=cust)
    r = hip.CustFragmentRunner(ctx, hip.to_device({k: fr.fact[k] for k in ("fk", "date", "price", "disc")}),
                               hip.to_device(fr.mid), fr.D, fr.k, key_bits=key_bits, cust_bits=cust_bits, gcap=cust,
                               join_cap=max(1, want["join_rows"]), revenue_bits=rbits, mid_sorted=mid == "sorted")
    assert "join_keyval" in _names(ctx, r.run)
    for _ in range(2):
        got = r.result()
        assert got["join_rows"] == want["join_rows"] and got["groups"] == want["groups"]
        for k in ("key", "sum", "cnt", "top_key", "top_sum", "top_cnt"):
            assert np.array_equal(got[k], want[k])
        r.run()
    assert ctx.errors() == 0


def _general(hip, fact, dim, fp, dp, group, aggs, key_bits, topk=0, vbits=0, labels=()):
    import torch
    ctx = hip.Context(0)
    want = oracle.fragment_general(fact, dim, fp, dp, 0, 0, group, aggs, topk=topk, gcap=1 << 20)
    dev = lambda cs: [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cs]
    fact, dim = dev(fact), dev(dim)
    box = {}

    def run():
        box["out"] = hip.fragment_run(ctx, fact, dim, fp, dp, 0, 0, group, aggs, topk=topk, key_bits=key_bits,
                                      gcap=max(1, want["groups"]), join_cap=max(1, want["join_rows"]), value_bits=vbits)
    names = _names(ctx, run)
    assert all(x in names for x in labels)
    out = box["out"]
    assert ctx.errors() == 0 and int(out["d_ngroups"]) == want["groups"] and int(out["d_join"]) == want["join_rows"]
    assert np.array_equal(out["key"][: want["groups"]].cpu().numpy(), want["key"])
    for a, b in zip(out["vals"], want["vals"]):
        assert np.array_equal(a[: want["groups"]].cpu().numpy().view(np.int64), np.asarray(b).view(np.int64))
    if topk:
        k = int(out["d_topk"])
        assert np.array_equal(out["top_key"][:k].cpu().numpy(), want["top_key"])
        assert np.array_equal(out["top_val"][:k].cpu().numpy(), want["top_val"])


REV = [(0, 2), (1, 100), (0, 3), (3, 0), (4, 0)]


@pytest.mark.parametrize("vbits", [0, 32])
@pytest.mark.parametrize("dup", [False, True])
def test_general_keyed(hip, vbits, dup):
    fr = datagen.config2(seed=12, n=400_000, m=100_000, cust_hi=70_000)
    pk = fr.mid["pk"] // 2 if dup else fr.mid["pk"]
    fact = [fr.fact[k] for k in ("fk", "date", "price", "disc")]
    _general(hip, fact, [pk, fr.mid["custkey"]], [(0, 1), (1, 2000), (8, 0)], [(0, 1), (1, 3), (6, 0), (1, 0), (13, 0)],
             [(5, 17)], [(1, [(0, 2), (1, 7), (3, 0)]), (0, [])], 0, topk=20, vbits=vbits,
             labels=("fragment_sort_fact", "fragment_join"))


@pytest.mark.parametrize("dup", [False, True])
def test_general_pairs(hip, dup):
    fact, dim = datagen.fact_table(77, 300_000, 9_000), datagen.dim_table(77, 9_000)
    pk = dim["pk"] // 3 if dup else dim["pk"]
    _general(hip, [fact[k] for k in ("fk", "date", "price", "disc", "flagA", "flagB")], [pk, dim["seg"]],
             [(0, 1), (1, 2400), (8, 0)], [(0, 1), (1, 1), (12, 0)], [(4, 2), (5, 1)],
             [(1, REV), (0, []), (4, [(0, 2)]), (2, [(0, 3)]), (3, [(0, 2)])], 0, topk=3,
             labels=("fragment_sort_fact", "fragment_join"))


def test_general_fact_order(hip):
    """16M fact rows whose columns outgrow the last-level cache: the joined pairs are sorted by fact row."""
    fact, dim = datagen.fact_table(4243, 16_000_000, 400_000), datagen.dim_table(4243, 400_000)
    _general(hip, [fact[k] for k in ("fk", "date", "price", "disc", "flagA", "flagB")], [dim["pk"], dim["seg"]],
             [(0, 1), (1, 2400), (8, 0)], [(0, 1), (1, 1), (12, 0)], [(4, 2), (5, 1)],
             [(1, REV), (0, []), (4, [(0, 2)]), (2, [(0, 3)]), (3, [(0, 2)])], 21, topk=3,
             labels=("fragment_sort_rows", "fragment_join"))


def test_server_undeclared_widths(hip):
    """A server whose widths are left at their default: flags alone and batched, and custkey requests."""
    t = datagen.config4_tables(seed=31, n=400_000, m_mid=100_000, m_dim=5_000, cust_hi=9_000)
    dev = {k: hip.to_device(t[k]) for k in ("fact", "mid", "dim")}
    reqs = datagen.config4_requests(9, 24, 400_000, p_cust=0.2, len_lo=1e3, len_hi=2e5)
    f = t["fact"]
    for slots, most in ((2, 8), (1, 1)):
        srv = hip.Server(dev, slots=slots, max_batch=most, max_flags_rows=200_000)
        for i, r in enumerate(reqs):
            srv.submit(0 if r["kind"] == "cust" else 1, r["D"], c=r["c"], k=100, row0=r["start"], n_rows=r["len"], tag=i)
        srv.drain()
        out = {r["tag"]: r for r in srv.poll()}
        srv.close()
        for i, r in enumerate(reqs):
            got = out[i]
            assert got["status"] == 0 and got["dev_errors"] == 0
            if r["kind"] == "cust":
                want = oracle.fragment_cust({k: f[k] for k in ("fk", "date", "price", "disc")}, t["mid"], r["D"], 100)
                assert got["join_rows"] == want["join_rows"] and got["top_key"] == want["top_key"].tolist()
                assert got["top_sum"] == want["top_sum"].tolist() and got["top_cnt"] == want["top_cnt"].tolist()
            else:
                sl = slice(r["start"], r["start"] + r["len"])
                fact = {k: f["fk_dim" if k == "fk" else k][sl] for k in ("fk", "date", "price", "disc", "flagA", "flagB")}
                want = oracle.fragment_flags(fact, t["dim"], r["D"], r["c"])
                assert got["join_rows"] == want["join_rows"] and got["key"] == want["key"].tolist()
                assert got["sum"] == want["sum"].tolist() and got["cnt"] == want["cnt"].tolist()
