"""Which flags fragments take the key table: not those of a context with its own digit width, nor a batch whose tables
would need much more scratch than its sorts, nor a call whose workspace fits the sorts alone."""
import ctypes

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


def _fragment(n, m, i=0):
    fr = datagen.random_flags_fragment(400 + i, n, m, m, 2000, i % 5)
    return fr, oracle.fragment_flags(fr.fact, fr.dim, fr.D, fr.c)


@pytest.mark.parametrize("digits", [4, 8, 11])
@pytest.mark.parametrize("n,m,key_bits", [(5_000, 900, 10), (60_000, 9_000, 14), (200_000, 40_000, 16)])
def test_digit_width(hip, n, m, key_bits, digits):
    """A digit width set by the caller asks for the sorts."""
    ctx = hip.Context(0)
    ctx.set_digit_bits(digits)
    fr, want = _fragment(n, m)
    run = hip.FlagsFragmentRunner(ctx, hip.to_device(fr.fact), hip.to_device(fr.dim), fr.D, fr.c, key_bits)
    names = _names(ctx, run.run)
    assert ("flags_fact" in names or "flags_fact_lds" in names) == (digits == 8)
    assert ("join_flags_agg" in names) == (digits != 8)
    for _ in range(2):
        run.run()
        _same(run.result(), want)
    b = hip.BatchRunner(ctx, [{"fact": run.fact, "dim": run.dim, "D": fr.D, "c": fr.c, "key_bits": key_bits}] * 2)
    assert ("batch_flags_fact" in _names(ctx, b.run)) == (digits == 8)
    for got in b.results():
        _same(got, want)
    assert ctx.errors() == 0
    b.close()


@pytest.mark.parametrize("count,table", [(12, True), (40, False)])
def test_batch_scratch(hip, count, table):
    """Small fragments over a declared domain of 2^18 keys: 1.1 MB of table each, up to 16 MB in all."""
    ctx = hip.Context(0)
    frags, wants = [], []
    for i in range(count):
        fr, want = _fragment(900 + i, 25, i)
        frags.append({"fact": hip.to_device(fr.fact), "dim": hip.to_device(fr.dim), "D": fr.D, "c": fr.c, "key_bits": 18})
        wants.append(want)
    b = hip.BatchRunner(ctx, frags)
    assert ("batch_flags_fact" in _names(ctx, b.run)) == table
    assert b.ws.numel() < 18 << 20
    for _ in range(2):
        b.run()
        for got, want in zip(b.results(), wants):
            _same(got, want)
    assert ctx.errors() == 0
    b.close()


def test_workspace_of_the_sorts(hip):
    """1,000 rows over 2^18 keys: the sorts need 38 KB, the table 1.1 MB.  A call with 256 KB is served."""
    import torch
    ctx = hip.Context(0)
    fr, want = _fragment(1_000, 25)
    run = hip.FlagsFragmentRunner(ctx, hip.to_device(fr.fact), hip.to_device(fr.dim), fr.D, fr.c, 18)
    assert "flags_fact" in _names(ctx, run.run)
    _same(run.result(), want)
    run.ws, run.ws_bytes = torch.empty(256 << 10, dtype=torch.uint8, device="cuda"), ctypes.c_size_t(256 << 10)
    for v in run.out.values():
        v.fill_(-1)
    assert "join_flags_agg" in _names(ctx, run.run)
    _same(run.result(), want)
    run.ws_bytes = ctypes.c_size_t(1 << 10)
    with pytest.raises(hip.TQPError):
        run.run()
    assert ctx.errors() == 0


def test_autotune_of_tables(hip):
    """A batch by tables has one launch sequence: autotune keeps the configuration."""
    ctx = hip.Context(0)
    fr, want = _fragment(20_000, 500)
    b = hip.BatchRunner(ctx, [{"fact": hip.to_device(fr.fact), "dim": hip.to_device(fr.dim), "D": fr.D, "c": fr.c,
                               "key_bits": 9}] * 3)
    for config in (1, 2):
        b.set_config(config)
        times = b.autotune(reps=2)
        assert b.config()[0] == config and len(set(times.values())) == 1 and min(times.values()) > 0
        for got in b.results():
            _same(got, want)
    b.close()
