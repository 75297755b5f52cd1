"""Dim sides with keys that many rows share, where an atomic per row takes turns on one word: the flags table, the
pair table and the join table against the oracle, at shares from one lane of a wave to all of them, and within the time that the rows'
own work takes."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu


def _keys(shape, m, r):
    pk = r.permutation(m)
    if shape == "half":
        pk[r.random(m) < 0.5] = 3
    elif shape == "tenth":
        pk[r.random(m) < 0.1] = 3
    elif shape == "all":
        pk[:] = 3
    elif shape == "runs":                            # 1 to 70 rows of a key, one after the other
        pk = np.repeat(np.arange(m), np.arange(m) % 70 + 1)[:m]
    elif shape == "twice":
        pk = pk // 2
    return pk.astype(np.int32)


@pytest.mark.parametrize("shape", ["half", "tenth", "all", "runs", "twice"])
@pytest.mark.parametrize("m,key_bits", [(63, 13), (5_000, 13), (70_001, 17)])
def test_flags(hip, m, key_bits, shape):
    ctx = hip.Context(0)
    r = np.random.default_rng(m)
    fr = datagen.random_flags_fragment(m % 89, 40_000, m, m, 2000, 1)
    dim = dict(fr.dim, pk=_keys(shape, m, r))
    want = oracle.fragment_flags(fr.fact, dim, fr.D, fr.c)
    fact, ddim = hip.to_device(fr.fact), hip.to_device(dim)
    one = hip.FlagsFragmentRunner(ctx, fact, ddim, fr.D, fr.c, key_bits)
    many = hip.BatchRunner(ctx, [{"fact": fact, "dim": ddim, "D": fr.D, "c": fr.c, "key_bits": key_bits}] * 3)
    for _ in range(2):
        one.run()
        many.run()
        for got in [one.result(), *many.results()]:
            assert got["join_rows"] == want["join_rows"]
            for k in ("key", "sum", "cnt"):
                assert np.array_equal(got[k], want[k])
    assert ctx.errors() == 0
    many.close()


@pytest.mark.parametrize("shape", ["half", "tenth", "runs", "twice"])
@pytest.mark.parametrize("n,m,key_bits", [(300, 63, 9), (20_000, 5_000, 13), (30_000, 70_001, 17)])
def test_pairs(hip, n, m, key_bits, shape):
    import torch
    ctx = hip.Context(0)
    r = np.random.default_rng(n)
    pk = _keys(shape, m, r)
    fk = r.integers(4, m, n).astype(np.int32)        # few meet the frequent key
    fk[:20] = 3
    fact = [fk, r.integers(-1000, 1000, n).astype(np.int32), r.integers(0, 4, n).astype(np.int8)]
    dim = [pk, r.integers(0, 3, m).astype(np.int32)]
    aggs = [(1, [(0, 1), (0, 4), (3, 0)]), (0, []), (2, [(0, 1)]), (3, [(0, 4)])]
    pred = [(0, 1), (1, 1), (12, 0)]                 # one of the dim rows' three values
    want = oracle.fragment_general(fact, dim, [], pred, 0, 0, [(2, 2), (4, 2)], aggs, topk=0, gcap=64)
    dev = lambda cs: [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cs]
    ctx.set_profiling(True)
    got = hip.fragment_run(ctx, dev(fact), dev(dim), [], pred, 0, 0, [(2, 2), (4, 2)], aggs, key_bits=key_bits, gcap=12,
                           join_cap=max(1, want["join_rows"]))
    assert "fragment_pairs" in [x for x, _ in ctx.profile_read()]
    g = int(got["d_ngroups"])
    assert ctx.errors() == 0 and g == want["groups"] and int(got["d_join"]) == want["join_rows"]
    assert np.array_equal(got["key"][:g].cpu().numpy(), want["key"])
    for a, b in zip(got["vals"], want["vals"]):
        assert np.array_equal(a[:g].cpu().numpy().view(np.int64), np.asarray(b).view(np.int64))


def _ms(ctx, label):
    return sum(t for n, t in ctx.profile_read() if n == label)


def test_flags_time(hip):
    """3M dim rows, half of them on one key: 0.27 ms; with an atomic per row 20."""
    import torch
    ctx = hip.Context(0)
    m = 3_000_000
    fr = datagen.random_flags_fragment(5, 1000, 1000, 1000, 2000, 1)
    pk = torch.randperm(m, device="cuda").to(torch.int32)
    pk[: m // 2] = 3
    dim = {"pk": pk[torch.randperm(m, device="cuda")].contiguous(), "seg": torch.ones(m, dtype=torch.int8, device="cuda")}
    run = hip.FlagsFragmentRunner(ctx, hip.to_device(fr.fact), dim, 2000, 1, 22)
    run.run()
    ctx.set_profiling(True)
    run.run()
    assert 0 < _ms(ctx, "flags_dim") < 3.0


def test_pairs_time(hip):
    """900k dim rows, half of them on one key: 0.35 ms; with an atomic per row 5.6."""
    import torch
    ctx = hip.Context(0)
    m = 900_000
    pk = torch.randperm(m, device="cuda").to(torch.int32)
    pk[: m // 2] = 3
    n = 1_000_000
    fact = [torch.full((n,), m, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int8, device="cuda")]
    args = (ctx, fact, [pk[torch.randperm(m, device="cuda")].contiguous()], [], [], 0, 0, [(1, 2)], [(0, [])])
    hip.fragment_run(*args, key_bits=20, gcap=4)
    ctx.set_profiling(True)
    hip.fragment_run(*args, key_bits=20, gcap=4)
    assert 0 < _ms(ctx, "fragment_pair_count") < 1.5


@pytest.mark.parametrize("shape", ["half", "tenth", "runs", "twice"])
@pytest.mark.parametrize("sorted_", [False, True])
@pytest.mark.parametrize("n,m,key_bits", [(20_000, 5_000, 13), (300_000, 70_001, 18), (3_000_000, 90_000, 21)])
def test_join_table(hip, n, m, key_bits, sorted_, shape):
    ctx = hip.Context(0)
    r = np.random.default_rng(n)
    pk, ck = _keys(shape, m, r), r.integers(0, 5000, m).astype(np.int32)
    if sorted_:
        o = np.argsort(pk, kind="stable")
        pk, ck = pk[o], ck[o]
    fk = r.integers(4, m, n).astype(np.int32)        # few meet the frequent key
    fk[:20] = 3
    fact = {"fk": fk, "date": r.integers(0, 100, n).astype(np.int32), "price": r.integers(1, 10_000, n),
            "disc": r.integers(0, 11, n)}
    mid = {"pk": pk, "custkey": ck}
    want = oracle.fragment_cust(fact, mid, 90, 10, gcap=5000)
    run = hip.CustFragmentRunner(ctx, hip.to_device(fact), hip.to_device(mid), 90, 10, key_bits=key_bits, cust_bits=13,
                                 gcap=5000, join_cap=max(n, want["join_rows"]), mid_sorted=sorted_)
    ctx.set_profiling(True)
    run.run()
    assert "probe" in [x for x, _ in ctx.profile_read()]
    got = run.result()
    assert ctx.errors() == 0 and got["join_rows"] == want["join_rows"] and got["groups"] == want["groups"]
    for k in ("key", "sum", "cnt", "top_key", "top_sum", "top_cnt"):
        assert np.array_equal(got[k], want[k])


def test_join_table_time(hip):
    """1.5M dim rows, half of them on one key: 1.16 ms to build; with an LDS atomic per row 1.94."""
    import torch
    ctx = hip.Context(0)
    n, m = 6_000_000, 1_500_000
    pk = torch.randperm(m, device="cuda").to(torch.int32)
    pk[: m // 2] = 0
    z = lambda t: torch.zeros(n, dtype=t, device="cuda")
    fact = {"fk": torch.randint(1, m, (n,), dtype=torch.int32, device="cuda"), "date": z(torch.int32),
            "price": z(torch.int64), "disc": z(torch.int64)}
    mid = {"pk": pk[torch.randperm(m, device="cuda")].contiguous(), "custkey": torch.zeros(m, dtype=torch.int32, device="cuda")}
    run = hip.CustFragmentRunner(ctx, fact, mid, 5, 10, key_bits=21, cust_bits=13, gcap=8192)
    run.run()
    ctx.set_profiling(True)
    run.run()
    assert 0 < _ms(ctx, "table_build") < 1.6
