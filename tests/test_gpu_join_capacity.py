"""Joins far larger than their capacity: a key that is frequent on both sides gives 2.8e9 pairs (more than the
chunk lists' 24-bit chunk numbers could count) and 1.2e12 (more than 40 bits).  The answer is the true size, the
capacity flag and exactly the capacity's rows, within a moment: pairs past the capacity are counted, not made."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _columns(n, m, key_bits, seed):
    """Fact key and the dim side, half of both on key 9, the rest on no common key."""
    r = np.random.default_rng(seed)
    fk, pk = r.integers(10, 1 << key_bits, n) | 1, r.integers(10, 1 << key_bits, m) & ~1
    fk[r.permutation(n)[: n // 2]] = 9
    pk[r.permutation(m)[: m // 2]] = 9
    return r, fk.astype(np.int32), pk.astype(np.int32), (n // 2) * (m // 2)


def _names(ctx):
    names = [k for k, _ in ctx.profile_read()]
    ctx.set_profiling(False)
    return names


@pytest.mark.parametrize("n,m,key_bits,cap", [(140_000, 80_000, 17, 3_000_001), (2_400_000, 2_000_000, 21, 3_000_001)])
@pytest.mark.parametrize("rbits", [32, 64])
def test_custkey(hip, n, m, key_bits, cap, rbits):
    ctx = hip.Context(0)
    r, fk, pk, pairs = _columns(n, m, key_bits, n)
    fact = {"fk": fk, "date": r.integers(0, 100, n).astype(np.int32), "price": r.integers(1, 1000, n),
            "disc": r.integers(0, 11, n)}
    mid = {"pk": pk, "custkey": r.integers(0, 5000, m).astype(np.int32)}
    run = hip.CustFragmentRunner(ctx, hip.to_device(fact), hip.to_device(mid), 100, 10, key_bits=key_bits,
                                 cust_bits=13, gcap=5000, join_cap=cap, revenue_bits=rbits)
    assert run.plan()["mid_passes"] == 1             # the key table
    for _ in range(2):
        ctx.set_profiling(True)
        run.run()
        assert "probe_lists" in _names(ctx)
        got = run.result()
        assert ctx.errors() == hip.DEVERR_CAPACITY
        assert got["join_rows"] == pairs and int(got["cnt"].sum()) == cap


@pytest.mark.parametrize("form", ["keyed", "pairs"])
def test_general(hip, form):
    """The keyed form (a 17-bit group column of the dim side) and the pairs (a group column of the fact side)."""
    import torch
    ctx = hip.Context(0)
    n, m, cap = 140_000, 80_000, 3_000_001
    r, fk, pk, pairs = _columns(n, m, 17, 7)
    dev = lambda cs: [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cs]
    fact = dev([fk, r.integers(0, 1000, n).astype(np.int32), r.integers(0, 4, n).astype(np.int32)])
    dim = dev([pk, r.integers(0, 70_000, m).astype(np.int32)])
    ctx.set_profiling(True)
    out = hip.fragment_run(ctx, fact, dim, [], [], 0, 0, [(4, 17)] if form == "keyed" else [(2, 2)],
                           [(1, [(0, 1)]), (0, [])], key_bits=17, gcap=70_000 if form == "keyed" else 4, join_cap=cap)
    assert ("fragment_probe_lists" if form == "keyed" else "fragment_pairs_long") in _names(ctx)
    assert ctx.errors() == hip.DEVERR_CAPACITY and int(out["d_join"]) == pairs
    assert int(out["vals"][1][: int(out["d_ngroups"])].sum()) == cap


def test_group_capacity_beyond_the_keys(hip):
    """A group capacity larger than the custkeys' domain: no more scratch than for the domain, whatever k."""
    ctx = hip.Context(0)
    r = np.random.default_rng(3)
    n, m = 300_000, 90_000
    fact = hip.to_device({"fk": r.integers(0, m, n).astype(np.int32), "date": r.integers(0, 100, n).astype(np.int32),
                          "price": r.integers(1, 1000, n), "disc": r.integers(0, 11, n)})
    mid = hip.to_device({"pk": r.permutation(m).astype(np.int32), "custkey": r.integers(0, 1 << 13, m).astype(np.int32)})
    runs = [hip.CustFragmentRunner(ctx, fact, mid, 90, 1000, key_bits=17, cust_bits=13, gcap=g << 13) for g in (1, 64)]
    assert all(x.plan()["mid_passes"] == 1 for x in runs) and runs[0].ws.numel() == runs[1].ws.numel()
    for x in runs:
        x.run()
    a, b = (x.result() for x in runs)
    assert ctx.errors() == 0 and all(np.array_equal(a[k], b[k]) for k in a)
