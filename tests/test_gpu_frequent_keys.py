"""Dim sides with keys that many rows share, where an atomic per row takes turns on one word: the flags table against
the oracle, at shares from one lane of a wave to all of them, and within the time that the rows' own work takes."""
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
