"""The hash group-by's per-block tables: rows at the edges of a block's step and of the grid, tables of 64 and
128 KB, and more groups than the capacity."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hip():
    return pytest.importorskip("paper_2203_01877_amd")


def _reference(key, val):
    u, inv = np.unique(key, return_inverse=True)
    o = np.argsort(inv, kind="stable")
    at = np.searchsorted(inv[o], np.arange(len(u)))
    v = val[o]
    return u, np.bincount(inv, minlength=len(u)), np.add.reduceat(v, at), np.minimum.reduceat(v, at), \
        np.maximum.reduceat(v, at)


@pytest.mark.parametrize("minmax", [False, True])
@pytest.mark.parametrize("n,g", [
    (1, 1), (4_095, 1), (4_096, 300), (4_097, 1_000),        # a block's step of rows
    (4_096 * 40 + 1, 3),                                     # several steps of a full grid
    ((1 << 21) - 1, 2_048), (1 << 21, 2_048),                # the table of 128 KB from here on
    (1 << 21, 2_049), ((1 << 21) + 17, 4_096),               # with sums and counts alone, up to 4096 groups
])
def test_hash_block_tables(hip, n, g, minmax):
    import torch
    ctx = hip.Context(0)
    r = np.random.default_rng(n + g)
    key = r.integers(0, g, n).astype(np.int32) * 7919
    val = r.integers(-(1 << 62), 1 << 62, n)
    u, cnt, sm, mn, mx = _reference(key, val)
    for _ in range(2):
        got = hip.hash_groupby(ctx, torch.from_numpy(key).cuda(), torch.from_numpy(val).cuda(), gcap=g, minmax=minmax)
        m = int(got["d_ngroups"])
        assert m == len(u) and ctx.errors() == 0
        o = np.argsort(got["key"][:m].cpu().numpy())
        col = lambda c: got[c][:m].cpu().numpy()[o]
        assert np.array_equal(col("key"), u) and np.array_equal(col("cnt"), cnt) and np.array_equal(col("sum"), sm)
        if minmax:
            assert np.array_equal(col("min"), mn) and np.array_equal(col("max"), mx)


def test_hash_block_tables_over_capacity(hip):
    """More groups than the capacity, at a table of 128 KB: flagged, and no row of an admitted group lost."""
    import torch
    ctx = hip.Context(0)
    n, g, cap = (1 << 21) + 3, 5_000, 1_500
    key = (np.arange(n) * 31 % g).astype(np.int32)
    got = hip.hash_groupby(ctx, torch.from_numpy(key).cuda(), torch.ones(n, dtype=torch.int64).cuda(), gcap=cap,
                           minmax=True)
    m = int(got["d_ngroups"])
    assert ctx.errors() & hip.DEVERR_CAPACITY
    m = min(m, cap)
    k, s, c = (got[x][:m].cpu().numpy() for x in ("key", "sum", "cnt"))
    assert len(np.unique(k)) == m and np.array_equal(s, c) and np.all(c <= np.bincount(key, minlength=g)[k])
