"""The hash group-by over inputs that do not fit what its grid and tables are sized for: far more groups than the
capacity."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _dev(*cols):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cols]


@pytest.mark.parametrize("minmax,cap", [(True, 1_000), (True, 2_048), (False, 2_000), (False, 4_096)])
def test_many_groups_over_capacity(hip, minmax, cap):
    """A hundred times more groups than the capacity: the flag, no row of an admitted group counted twice, and no
    row that walks all slots of a full table (a launch of 2M rows then took 15 to 40 ms)."""
    ctx = hip.Context(0)
    n, g = (1 << 21) + 3, 400_000
    key = (np.arange(n, dtype=np.int64) * 7919 % g).astype(np.int32)
    k, one = _dev(key, np.ones(n, dtype=np.int64))
    for _ in range(2):
        ctx.set_profiling(True)
        got = hip.hash_groupby(ctx, k, one, gcap=cap, minmax=minmax)
        ms = sum(t for _, t in ctx.profile_read())
        ctx.set_profiling(False)
        assert ctx.errors() & hip.DEVERR_CAPACITY
    m = min(int(got["d_ngroups"]), cap)
    kk, s, c = (got[x][:m].cpu().numpy() for x in ("key", "sum", "cnt"))
    assert len(np.unique(kk)) == m and np.array_equal(s, c) and np.all(c <= np.bincount(key, minlength=g)[kk])
    assert ms < 10.0


def _groups(shape, n, r):
    lane = np.arange(n) % 64
    if shape == "one":
        return np.full(n, 5)
    if shape == "skew":                              # 90% of the rows on one group
        return np.where(r.random(n) < 0.9, 77, r.integers(0, 900, n))
    if shape == "half":                              # 32 lanes of a wave on the group of its first row
        return np.where(lane % 2 == 0, 3, 4 + lane)
    if shape == "less":                              # 31 lanes: one by one
        return np.where((lane % 2 == 0) & (lane != 62), 3, 4 + lane)
    return np.where(r.random(n) < 0.5, -1, 6)        # negative keys left out, some in a wave's first row


@pytest.mark.parametrize("n", [1, 63, 4_097, 100_003])
@pytest.mark.parametrize("shape", ["one", "skew", "half", "less", "negative"])
@pytest.mark.parametrize("cols", ["count", "sum", "minmax", "distinct"])
def test_rows_of_one_group(hip, n, shape, cols):
    """Waves whose lanes share a group, every set of columns, values up to the ends of int64."""
    ctx = hip.Context(0)
    r = np.random.default_rng(n)
    key = _groups(shape, n, r).astype(np.int32)
    val = r.integers(-(1 << 62), 1 << 62, n)
    val[:: 7], val[3:: 11] = np.iinfo(np.int64).min, np.iinfo(np.int64).max
    d = r.integers(0, 9, n).astype(np.int32)
    k, v, dv = _dev(key, val, d)
    got = hip.hash_groupby(ctx, k, v if cols != "count" else None, dval=dv if cols == "distinct" else None, gcap=1000,
                           minmax=cols in ("minmax", "distinct"))
    keep = key >= 0
    assert ctx.errors() == (0 if keep.all() else hip.DEVERR_KEY_RANGE)
    key, val, d = key[keep], val[keep], d[keep]
    u, inv = np.unique(key, return_inverse=True)
    m = int(got["d_ngroups"])
    o = np.argsort(got["key"][:m].cpu().numpy())
    col = lambda c: got[c][:m].cpu().numpy()[o]
    assert np.array_equal(col("key"), u) and np.array_equal(col("cnt"), np.bincount(inv, minlength=len(u)))
    if cols != "count":
        with np.errstate(over="ignore"):
            assert np.array_equal(col("sum"), np.array([val[inv == i].sum() for i in range(len(u))], dtype=np.int64))
    if cols in ("minmax", "distinct"):
        assert np.array_equal(col("min"), np.array([val[inv == i].min() for i in range(len(u))], dtype=np.int64))
        assert np.array_equal(col("max"), np.array([val[inv == i].max() for i in range(len(u))], dtype=np.int64))
    if cols == "distinct":
        assert np.array_equal(col("ndist"), np.array([len(np.unique(d[inv == i])) for i in range(len(u))]))


@pytest.mark.parametrize("n,g", [(200_000, 1_000), (1_000_000, 2_000), (1_000_000, 65), (300_001, 64)])
@pytest.mark.parametrize("cols", ["distinct", "sum", "minmax"])
def test_distinct_grid(hip, n, g, cols):
    """COUNT(DISTINCT) with few rows per group: the grid of the rows' own work, every row in one block."""
    ctx = hip.Context(0)
    r = np.random.default_rng(g)
    key, val, d = r.integers(0, g, n), r.integers(-1000, 1000, n), r.integers(0, 5000, n)
    k, v, dv = _dev(key.astype(np.int32), val, d.astype(np.int32))
    got = hip.hash_groupby(ctx, k, None if cols == "distinct" else v, dval=dv, gcap=g, minmax=cols == "minmax")
    m = int(got["d_ngroups"])
    assert m == len(np.unique(key)) and ctx.errors() == 0
    o = np.argsort(got["key"][:m].cpu().numpy())
    col = lambda c: got[c][:m].cpu().numpy()[o]
    assert np.array_equal(col("cnt"), np.bincount(key, minlength=g))
    assert np.array_equal(col("ndist"), np.bincount(np.unique(key * 5000 + d) // 5000, minlength=g))
    if cols != "distinct":
        assert np.array_equal(col("sum"), np.bincount(key, weights=val, minlength=g).astype(np.int64))


@pytest.mark.parametrize("minmax,g", [(False, 2_049), (True, 1_025)])
@pytest.mark.parametrize("less", [0, 1])
def test_large_table_rule(hip, minmax, g, less):
    """The first row count per group at which a table of 128 KB takes the rows, and one row fewer."""
    ctx = hip.Context(0)
    n = 2048 * g - less
    r = np.random.default_rng(g)
    key, val = r.integers(0, g, n), r.integers(-1000, 1000, n)
    k, v = _dev(key.astype(np.int32), val)
    ctx.set_profiling(True)
    got = hip.hash_groupby(ctx, k, v, gcap=g, minmax=minmax)
    assert ("hashagg_local" in [x for x, _ in ctx.profile_read()]) == (less == 0)
    m = int(got["d_ngroups"])
    o = np.argsort(got["key"][:m].cpu().numpy())
    assert m == g and ctx.errors() == 0
    assert np.array_equal(got["cnt"][:m].cpu().numpy()[o], np.bincount(key, minlength=g))
    assert np.array_equal(got["sum"][:m].cpu().numpy()[o], np.bincount(key, weights=val, minlength=g).astype(np.int64))
