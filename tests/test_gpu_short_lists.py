"""The probe of the join table over keys with a few dim rows each, expanded in rounds from 2^22 fact rows on: lists of
one length, of all lengths, and too few of them for a round; against the oracle, by both probe kernels."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

ROWS = 1 << 22


def _lengths(shape, keys, r):
    if isinstance(shape, int):
        return np.full(keys, shape)
    if shape == "all":                               # 0 to 6 rows of a key
        return r.integers(0, 7, keys)
    if shape == "few":                               # 3% of the keys twice
        return 1 + (r.random(keys) < 0.03)
    return np.where(np.arange(keys) < keys // 4, 2, np.where(np.arange(keys) < keys // 2, 9, 1))     # "parts"


def _case(n, key_bits, shape, seed=1):
    r = np.random.default_rng(seed)
    keys = 3 << (key_bits - 2)
    rows = np.repeat(np.arange(keys), _lengths(shape, keys, r))
    pk = rows[r.permutation(len(rows))].astype(np.int32)
    fact = {"fk": r.integers(0, 1 << key_bits, n).astype(np.int32), "date": r.integers(0, 100, n).astype(np.int32),
            "price": r.integers(90_000, 10_500_000, n), "disc": r.integers(0, 11, n)}
    return fact, {"pk": pk, "custkey": r.integers(0, 70_000, len(pk)).astype(np.int32)}


def _run(hip, ctx, fact, mid, key_bits, rbits, D, cap):
    run = hip.CustFragmentRunner(ctx, hip.to_device(fact), hip.to_device(mid), D, 20, key_bits=key_bits, cust_bits=17,
                                 gcap=70_000, join_cap=cap, revenue_bits=rbits)
    ctx.set_profiling(True)
    run.run()
    names = [k for k, _ in ctx.profile_read()]
    ctx.set_profiling(False)
    assert "probe" in names and ("probe_short" in names) == (len(fact["fk"]) >= ROWS)
    return run.result()


@pytest.mark.parametrize("rbits", [32, 64])
@pytest.mark.parametrize("shape", [1, 2, 3, 4, 5, "all", "few", "parts"])
@pytest.mark.parametrize("key_bits,n", [(17, ROWS), (21, ROWS + 4099)])
def test_rounds(hip, key_bits, n, shape, rbits):
    ctx = hip.Context(0)
    fact, mid = _case(n, key_bits, shape)
    want = oracle.fragment_cust(fact, mid, 70, 20, gcap=70_000)
    got = _run(hip, ctx, fact, mid, key_bits, rbits, 70, max(2 * n, want["join_rows"]))
    assert ctx.errors() == 0 and got["join_rows"] == want["join_rows"] and got["groups"] == want["groups"]
    for k in ("key", "sum", "cnt", "top_key", "top_sum", "top_cnt"):
        assert np.array_equal(got[k], want[k])


@pytest.mark.parametrize("n", [ROWS - 1, ROWS])
def test_rounds_capacity_and_range(hip, n):
    """Less room than pairs: the true size and exactly the capacity's rows.  A custkey outside its width on the
    second of a key's rows: flagged."""
    ctx = hip.Context(0)
    fact, mid = _case(n, 17, 3)
    want = oracle.fragment_cust(fact, mid, 70, 20, gcap=70_000)["join_rows"]
    for cap in (want - 1, n // 2):
        got = _run(hip, ctx, fact, mid, 17, 32, 70, cap)
        assert ctx.errors() == hip.DEVERR_CAPACITY and got["join_rows"] == want and int(got["cnt"].sum()) == cap
    mid["custkey"][np.flatnonzero(mid["pk"] == 77)[1]] = 1 << 17
    _run(hip, ctx, fact, mid, 17, 32, 70, want)
    assert ctx.errors() == hip.DEVERR_KEY_RANGE
