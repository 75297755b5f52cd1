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
