"""Cases that stand for the work a user of the library has it do, each through its public entry points.

A case is one query or one chain of operators over columns that are resident on the GPU.  The sizes are
those of bench.py and datagen (60k, 6M and 60M fact rows, dimension tables a fortieth of the fact table,
a mid table a quarter of it, 8M-row joins, batches of fragments of 1e3 to 4e6 rows) with ragged ones
between them.  Columns follow datagen's recipe: uniform foreign keys, shuffled primary keys, dates over
seven years, prices in cents, discounts in percent.  Every output a pass returns is written in full by the
library, or lies in a buffer that prepare() has cleared, so that the same inputs give the same outputs."""
import math

import torch

import paper_2203_01877_amd as tqp
from paper_2203_01877_amd import _lib

DAYS = 2557
_CTX = {}


def _ctx():
    """One context per process, as a program keeps one."""
    if "c" not in _CTX:
        _CTX["c"] = tqp.Context(0)
    return _CTX["c"]


# ---------------------------------------------------------------------------------------------- cases
def listed():
    return [
        # a dashboard's query over a small table: launches and latency are all there is
        {"name": "flags_60k", "kind": "flags", "n": 60_000, "m": 1_500, "D": 2400, "c": 1},
        # the same query over a table of ordinary size
        {"name": "flags_6m", "kind": "flags", "n": 6_000_000, "m": 150_000, "D": 2400, "c": 1},
        # the benchmark's query: revenue per customer and the top 100, revenue declared 32-bit
        {"name": "cust_60m", "kind": "cust", "n": 60_000_000, "m": 15_000_000, "cust": 1_500_000, "D": 2400,
         "k": 100, "rbits": 32, "miss": 0.2},
        # a ragged smaller one with a selective date and 64-bit revenue
        {"name": "cust_3m_ragged", "kind": "cust", "n": 3_000_017, "m": 750_003, "cust": 75_001, "D": 1000,
         "k": 10, "rbits": 0, "miss": 0.2},
        # the same kind of query written as a descriptor (joins, programs, top-k composed by the caller)
        {"name": "general_cust_24m", "kind": "gcust", "n": 24_000_000, "m": 6_000_000, "cust": 600_000, "D": 2400,
         "k": 100, "vbits": 0},
        # a report with few groups and every aggregate, as a descriptor, over a ragged table
        {"name": "general_flags_6m", "kind": "gflags", "n": 5_999_993, "m": 149_999, "D": 2400, "c": 1},
        # many users' small queries in one launch sequence
        {"name": "batch_64", "kind": "batch", "nf": 64, "lo": 1_000, "hi": 4_000_000, "mixseed": 3},
        # operators composed by hand: sort both sides, join, read columns through the row positions
        {"name": "join_8m", "kind": "join", "n": 8_000_000, "m": 2_000_000},
        # a plan of three joins and the revenue per customer over its tuples
        {"name": "chain_20m", "kind": "chain", "n": 20_000_000, "m": 5_000_000, "cust": 500_000, "nation": 25,
         "dense": True},
        # a group-by over many groups, sort-based (the result comes in key order)
        {"name": "groupby_40m", "kind": "groupby", "n": 40_000_000, "g": 1_500_000, "avg": False},
        # a group-by over few groups, hash-based, every statistic, then ORDER BY key
        {"name": "hash_groupby_30m", "kind": "hashgb", "n": 30_000_000, "g": 1_000},
        # a scan: a computed column and a filter over it that carries a column along
        {"name": "scan_60m", "kind": "scan", "n": 60_000_000, "D": 1200},
    ]


def _log(rng, lo, hi):
    """A size between lo and hi, even over the logarithm; most are odd or ragged."""
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["flags", "cust", "gcust", "gflags", "batch", "join", "chain", "groupby", "hashgb", "scan"])
    if kind in ("flags", "gflags"):
        n = _log(rng, 20_000, 12_000_000)
        return {"kind": kind, "n": n, "m": max(500, n // rng.choice([20, 40, 80])), "D": rng.choice([100, 1000, 2400, 2557]),
                "c": rng.randrange(5)}
    if kind == "cust":
        n = _log(rng, 100_000, 50_000_000)
        m = n // rng.choice([3, 4, 8])
        return {"kind": kind, "n": n, "m": m, "cust": max(100, m // 10), "D": rng.choice([100, 1000, 2400]),
                "k": rng.choice([1, 10, 100]), "rbits": rng.choice([0, 32]), "miss": rng.choice([0.0, 0.2])}
    if kind == "gcust":
        n = _log(rng, 100_000, 24_000_000)
        m = n // rng.choice([4, 6])
        return {"kind": kind, "n": n, "m": m, "cust": max(100, m // 10), "D": rng.choice([2000, 2400]),
                "k": rng.choice([1, 10, 100]), "vbits": rng.choice([0, 32])}
    if kind == "batch":
        return {"kind": kind, "nf": rng.randrange(8, 65), "lo": 1_000, "hi": _log(rng, 100_000, 4_000_000),
                "mixseed": rng.randrange(1000)}
    if kind == "join":
        n = _log(rng, 50_000, 12_000_000)
        return {"kind": kind, "n": n, "m": max(100, n // rng.choice([1, 4, 40]))}
    if kind == "chain":
        n = _log(rng, 100_000, 20_000_000)
        return {"kind": kind, "n": n, "m": n // 4, "cust": n // 40, "nation": 25, "dense": rng.random() < 0.5}
    if kind == "groupby":
        n = _log(rng, 50_000, 40_000_000)
        return {"kind": kind, "n": n, "g": _log(rng, 5, max(6, n // 20)), "avg": n < 15_000_000 and rng.random() < 0.5}
    if kind == "hashgb":
        n = _log(rng, 50_000, 30_000_000)
        return {"kind": kind, "n": n, "g": _log(rng, 5, max(6, n // 20))}
    return {"kind": kind, "n": _log(rng, 50_000, 60_000_000), "D": rng.choice([100, 1200, 2400])}


# ---------------------------------------------------------------------------------------------- inputs
class _Draws:
    """Columns on the GPU, made from the seed alone."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1_000_003 * int(seed) + 20220301)

    def ints(self, n, lo, hi, dtype=torch.int32):
        return torch.randint(lo, hi, (n,), generator=self.g, dtype=dtype, device="cuda")

    def perm(self, n):
        return torch.randperm(n, generator=self.g, dtype=torch.int64, device="cuda").to(torch.int32)

    def covering(self, n, hi):
        """n values of [0, hi), each value at least once (n >= hi), in random order."""
        v = self.ints(n, 0, hi)
        v[self.perm(n)[:hi].long()] = torch.arange(hi, dtype=torch.int32, device="cuda")
        return v

    def fact(self, n, fk_hi):
        return {"fk": self.ints(n, 0, fk_hi), "date": self.ints(n, 0, DAYS),
                "price": self.ints(n, 90_000, 10_500_000, torch.int64), "disc": self.ints(n, 0, 11, torch.int64),
                "flagA": self.ints(n, 0, 3, torch.int8), "flagB": self.ints(n, 0, 2, torch.int8)}

    def dim(self, m):
        return {"pk": self.perm(m), "seg": self.ints(m, 0, 5, torch.int8)}


def _bits(values):
    """Width of the values 0 .. values - 1."""
    return max(1, int(values - 1).bit_length())


def _batch_sizes(case):
    """Fact rows of each fragment of a batch, even over the logarithm."""
    out, x = [], int(case["mixseed"]) * 2654435761 % 2**32
    for _ in range(int(case["nf"])):
        x = (x * 1664525 + 1013904223) % 2**32
        out.append(int(math.exp(math.log(case["lo"]) + (x / 2**32) * (math.log(case["hi"]) - math.log(case["lo"])))))
    return out


def _columns(case, seed):
    """The tables of a case."""
    d, kind = _Draws(seed), case["kind"]
    if kind in ("flags", "gflags"):
        return {"fact": d.fact(case["n"], case["m"]), "dim": d.dim(case["m"])}
    if kind in ("cust", "gcust"):
        m = case["m"]
        hi = m + int(m * case.get("miss", 0.0) / (1 - case.get("miss", 0.0)))
        f = d.fact(case["n"], hi)
        return {"fact": f, "mid": {"pk": d.perm(m), "custkey": d.perm(m) % case["cust"]}, "fk_hi": hi}
    if kind == "batch":
        fr = []
        for i, n in enumerate(_batch_sizes(case)):
            m = max(1, n // 40)
            fr.append({"fact": d.fact(n, m), "dim": d.dim(m), "D": (997 * i) % DAYS, "c": i % 5, "key_bits": _bits(m)})
        return {"fragments": fr}
    if kind == "join":
        n, m = case["n"], case["m"]
        return {"lkey": d.ints(n, 0, m), "price": d.ints(n, 90_000, 10_500_000, torch.int64), "rkey": d.perm(m),
                "attr": d.ints(m, 0, 1 << 20)}
    if kind == "chain":
        n, m, c, k = case["n"], case["m"], case["cust"], case["nation"]
        ar = lambda v: torch.arange(v, dtype=torch.int32, device="cuda")
        return {"fk": d.covering(n, m), "price": d.ints(n, 90_000, 10_500_000, torch.int64), "mid_pk": ar(m),
                "mid_cust": d.covering(m, c), "cust_pk": d.perm(c), "cust_nation": d.ints(c, 0, k), "nation_pk": ar(k)}
    if kind == "groupby":
        t = {"key": d.covering(case["n"], case["g"]), "val": d.ints(case["n"], -(1 << 40), 1 << 40, torch.int64)}
        if case["avg"]:
            t["avg"] = d.ints(case["n"], 90_000, 10_500_000, torch.int64)
        return t
    if kind == "hashgb":
        return {"key": d.covering(case["n"], case["g"]), "val": d.ints(case["n"], -(1 << 40), 1 << 40, torch.int64)}
    n = case["n"]
    return {"date": d.ints(n, 0, DAYS), "price": d.ints(n, 90_000, 10_500_000, torch.int64),
            "disc": d.ints(n, 0, 11, torch.int64), "flag": d.ints(n, 0, 3, torch.int8), "fk": d.ints(n, 0, max(1, n // 4))}


# programs over (fk, date, price, disc, flagA, flagB): price * (100 - disc), date < D
def _revenue(price, disc):
    return [(0, price), (1, 100), (0, disc), (3, 0), (4, 0)]


def _less(col, d):
    return [(0, col), (1, d), (8, 0)]


def _scan_program(case):
    """CASE WHEN date < D THEN price * (100 - disc) ELSE 0 END + flag, over (date, price, disc, flag)."""
    return _less(0, case["D"]) + _revenue(1, 2) + [(1, 0), (17, 0), (0, 3), (2, 0)]


def prepare(case, seed):
    case, ctx, kind = dict(case), _ctx(), case["kind"]
    t = _columns(case, seed)
    s = {"case": case, "ctx": ctx, "t": t}
    if kind == "flags":
        s["run"] = tqp.FlagsFragmentRunner(ctx, t["fact"], t["dim"], case["D"], case["c"], key_bits=_bits(case["m"]))
    elif kind == "cust":
        s["run"] = tqp.CustFragmentRunner(ctx, t["fact"], t["mid"], case["D"], k=case["k"], key_bits=_bits(t["fk_hi"]),
                                          cust_bits=_bits(case["cust"]), gcap=case["cust"], revenue_bits=case["rbits"])
    elif kind == "batch":
        s["run"] = tqp.BatchRunner(ctx, t["fragments"])
    elif kind == "scan":
        n = case["n"]
        s["row"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        s["carried"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    if "run" in s:
        for v in s["run"].out.values():
            v.zero_()
    return s


# ---------------------------------------------------------------------------------------------- one pass
def run(s):
    case, ctx, t = s["case"], s["ctx"], s["t"]
    kind = case["kind"]
    if kind in ("flags", "cust", "batch"):
        s["run"].run()
        return s["run"].out
    if kind == "gcust":
        f, m = t["fact"], t["mid"]
        return tqp.fragment_run(ctx, [f["fk"], f["date"], f["price"], f["disc"]], [m["pk"], m["custkey"]],
                                _less(1, case["D"]), [], 0, 0, [(5, _bits(case["cust"]))],
                                [(_lib.AGG_SUM, _revenue(2, 3)), (_lib.AGG_COUNT, [])], topk=case["k"],
                                key_bits=_bits(t["fk_hi"]), gcap=case["cust"], value_bits=case["vbits"])
    if kind == "gflags":
        f, d = t["fact"], t["dim"]
        price = [(0, 2)]
        r = tqp.fragment_run(ctx, [f["fk"], f["date"], f["price"], f["disc"], f["flagA"], f["flagB"]],
                             [d["pk"], d["seg"]], _less(1, case["D"]), [(0, 1), (1, case["c"]), (12, 0)], 0, 0,
                             [(4, 2), (5, 1)],
                             [(_lib.AGG_SUM, _revenue(2, 3)), (_lib.AGG_COUNT, []), (_lib.AGG_AVG, price),
                              (_lib.AGG_MIN, price), (_lib.AGG_MAX, price)], key_bits=_bits(case["m"]), gcap=6)
        return {"key": r["key"], "vals": r["vals"], "d_ngroups": r["d_ngroups"], "d_join": r["d_join"]}
    if kind == "join":
        kb = _bits(case["m"])
        lk, lrow = tqp.sort(ctx, t["lkey"], perm=True, key_bits=kb)
        rk, rrow = tqp.sort(ctx, t["rkey"], perm=True, key_bits=kb)
        ol, orr, cnt = tqp.join(ctx, lk, rk, lrow, rrow)
        return {"l": ol, "r": orr, "count": cnt, "price": tqp.gather(ctx, t["price"], ol),
                "attr": tqp.gather(ctx, t["attr"], orr)}
    if kind == "chain":
        dense = case["dense"]
        rows, j = tqp.join_chain(ctx, [t["fk"], t["mid_cust"], t["cust_nation"]],
                                 [t["mid_pk"], t["cust_pk"], t["nation_pk"]], pk_sorted=[True, False, True],
                                 key_bits=[_bits(case["m"]), _bits(case["cust"]), _bits(case["nation"])],
                                 pk_dense=[dense, False, dense])
        price = tqp.gather(ctx, t["price"], rows[0])
        return tqp.groupby_agg(ctx, rows[2], price, key_bits=_bits(case["cust"]), gcap=case["cust"])
    if kind == "groupby":
        return tqp.groupby_agg(ctx, t["key"], t["val"], t.get("avg"), key_bits=_bits(case["g"]), gcap=case["g"])
    if kind == "hashgb":
        r = tqp.hash_groupby(ctx, t["key"], t["val"], gcap=case["g"], minmax=True)
        key, p = tqp.sort(ctx, r["key"], perm=True, key_bits=_bits(case["g"]))
        return {"key": key, **{c: tqp.gather(ctx, r[c], p) for c in ("cnt", "sum", "min", "max")},
                "d_ngroups": r["d_ngroups"]}
    v = tqp.eval_expr(ctx, [t["date"], t["price"], t["disc"], t["flag"]], _scan_program(case))
    tqp.filter_noalloc(ctx, [t["date"], v], [(0, tqp.TQP_LT, case["D"]), (1, tqp.TQP_GT, 500_000_000)], s["row"],
                       s["count"], carry=t["fk"], out_carry=s["carried"])
    return {"value": v, "row": s["row"], "carried": s["carried"], "count": s["count"]}


# ---------------------------------------------------------------------------------------------- floors
def work(case):
    """Bytes of each referenced column read once and each result written once; a row the date filter drops
    still costs its key and date, the price, discount and flags of dropped rows do not count.  The
    operations are the comparisons, products and sums of the query, a handful per row."""
    kind, n = case["kind"], case.get("n", 0)
    if kind in ("flags", "gflags"):
        kept = n * min(1.0, case["D"] / DAYS)
        return {"bytes": 8 * n + 18 * kept / 5 + 5 * case["m"] + 300, "flops": 6 * n}
    if kind in ("cust", "gcust"):
        kept = n * min(1.0, case["D"] / DAYS) * (1 - case.get("miss", 0.0))
        return {"bytes": 8 * n + 16 * kept + 8 * case["m"] + 20 * case["cust"] + 20 * case["k"], "flops": 6 * n}
    if kind == "batch":
        b = f = 0
        for i, x in enumerate(_batch_sizes(case)):
            b += 8 * x + 18 * x * ((997 * i) % DAYS) / DAYS / 5 + 5 * (x // 40) + 300
            f += 6 * x
        return {"bytes": b, "flops": f}
    if kind == "join":
        return {"bytes": (4 + 8 + 4 + 4 + 8 + 4) * n + 8 * case["m"], "flops": 2 * n}
    if kind == "chain":
        return {"bytes": 12 * n + 8 * case["m"] + 28 * case["cust"], "flops": 4 * n}
    if kind in ("groupby", "hashgb"):
        col = 12 + (8 if case.get("avg") else 0)
        return {"bytes": col * n + (36 if kind == "hashgb" else 20 + (8 if case.get("avg") else 0)) * case["g"],
                "flops": 2 * n}
    kept = n * case["D"] / DAYS * 0.4
    return {"bytes": (4 + 8 + 8 + 1 + 8) * n + 12 * kept, "flops": 8 * n}


# ---------------------------------------------------------------------------------------------- exact values
def _group_sums(key, g, *cols):
    """Per group of [0, g): the sums of the columns, over a sort so that few groups do not serialise."""
    k, p = torch.sort(key.long())
    ends = torch.cumsum(torch.bincount(k, minlength=g), 0)
    out = []
    for c in cols:
        cs = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(c.long()[p], 0)])
        hi = cs[ends]
        out.append(hi - torch.cat([cs[:1], hi[:-1]]))
    return out


def _packed(present, *cols):
    """Rows of the groups that exist, first, and zeros behind them."""
    idx = torch.nonzero(present).reshape(-1)
    out = []
    for c in cols:
        z = torch.zeros_like(c)
        z[:idx.numel()] = c[idx]
        out.append(z)
    return out


def _top(key, val, k):
    v, p = torch.sort(val, descending=True, stable=True)
    return key[p][:k], v[:k], p[:k]


def _flags_exact(fact, dim, D, c):
    hit = torch.zeros(int(max(int(dim["pk"].max()), int(fact["fk"].max()))) + 1, dtype=torch.bool, device="cuda")
    hit[dim["pk"][dim["seg"] == c].long()] = True
    ok = (fact["date"] < D) & hit[fact["fk"].long()]
    g = fact["flagA"][ok].long() * 2 + fact["flagB"][ok].long()
    price = fact["price"][ok]
    rev, sp = _group_sums(g, 6, price * (100 - fact["disc"][ok]), price)
    return g, price, rev, sp, torch.bincount(g, minlength=6)


def exact(case, seed):
    t, kind = _columns(case, seed), case["kind"]
    one = lambda v: torch.tensor([int(v)], dtype=torch.int64, device="cuda")
    ar = lambda v: torch.arange(v, dtype=torch.int64, device="cuda")
    if kind in ("flags", "batch"):
        rows = []
        frs = t["fragments"] if kind == "batch" else [{**t, "D": case["D"], "c": case["c"]}]
        for fr in frs:
            g, _, rev, sp, cnt = _flags_exact(fr["fact"], fr["dim"], fr["D"], fr["c"])
            avg = sp.double() / cnt.clamp(min=1).double()
            key, s, n, a = _packed(cnt > 0, ar(6), rev, cnt, avg)
            two = lambda v: torch.cat([v, torch.zeros(2, dtype=v.dtype, device="cuda")])
            rows.append({"key": two(key).to(torch.int32), "sum": two(s), "cnt": two(n), "avg": two(a),
                         "d_ngroups": one((cnt > 0).sum()), "d_join": one(cnt.sum())})
        if kind == "flags":
            return rows[0]
        return {k: torch.cat([r[k] for r in rows]) if k.startswith("d_") else torch.stack([r[k] for r in rows])
                for k in rows[0]}
    if kind == "gflags":
        g, price, rev, sp, cnt = _flags_exact(t["fact"], t["dim"], case["D"], case["c"])
        if int((cnt > 0).sum()) < 6:
            return None
        lo = torch.stack([price[g == k].min() for k in range(6)])
        hi = torch.stack([price[g == k].max() for k in range(6)])
        return {"key": ar(6).to(torch.int32), "vals": [rev, cnt, sp.double() / cnt.double(), lo, hi],
                "d_ngroups": one(6), "d_join": one(cnt.sum())}
    if kind in ("cust", "gcust"):
        f, m, G = t["fact"], t["mid"], case["cust"]
        cust = torch.full((t["fk_hi"],), -1, dtype=torch.int64, device="cuda")
        cust[m["pk"].long()] = m["custkey"].long()
        key = cust[f["fk"].long()]
        ok = (f["date"] < case["D"]) & (key >= 0)
        s, = _group_sums(key[ok], G, f["price"][ok] * (100 - f["disc"][ok]))
        cnt = torch.bincount(key[ok], minlength=G)
        pk, ps, pc = _packed(cnt > 0, ar(G), s, cnt)
        ng, k = int((cnt > 0).sum()), case["k"]
        if ng < k or (kind == "gcust" and ng < G):
            return None
        tk, tv, tp = _top(pk[:ng], ps[:ng], k)
        if kind == "cust":
            return {"key": pk.to(torch.int32), "sum": ps, "cnt": pc, "d_ngroups": one(ng), "d_join": one(ok.sum()),
                    "top_key": tk.to(torch.int32), "top_sum": tv, "top_cnt": pc[:ng][tp],
                    "d_topk": one(k).to(torch.int32)}
        return {"key": pk.to(torch.int32), "vals": [ps, pc], "d_ngroups": one(ng), "d_join": one(ok.sum()),
                "top_key": tk.to(torch.int32), "top_val": tv, "d_topk": one(k).to(torch.int32)}
    if kind == "join":
        _, l = torch.sort(t["lkey"], stable=True)
        where = torch.empty(case["m"], dtype=torch.int64, device="cuda")
        where[t["rkey"].long()] = ar(case["m"])
        r = where[t["lkey"][l].long()]
        return {"l": l.to(torch.int32), "r": r.to(torch.int32), "count": one(case["n"]), "price": t["price"][l],
                "attr": t["attr"][r]}
    if kind == "chain":
        where = torch.empty(case["cust"], dtype=torch.int64, device="cuda")
        where[t["cust_pk"].long()] = ar(case["cust"])
        g = where[t["mid_cust"].long()[t["fk"].long()]]
        s, = _group_sums(g, case["cust"], t["price"])
        return {"key": ar(case["cust"]).to(torch.int32), "sum": s, "cnt": torch.bincount(g, minlength=case["cust"]),
                "avg": None, "d_ngroups": one(case["cust"])}
    if kind in ("groupby", "hashgb"):
        g = case["g"]
        cnt = torch.bincount(t["key"].long(), minlength=g)
        s, = _group_sums(t["key"], g, t["val"])
        out = {"key": ar(g).to(torch.int32), "sum": s, "cnt": cnt, "d_ngroups": one(g)}
        if kind == "hashgb":
            # sorted by (key, value): the first and the last row of each group
            v, p = torch.sort(t["val"])
            k, q = torch.sort(t["key"][p], stable=True)
            v, ends = v[q], torch.cumsum(cnt, 0)
            out["min"], out["max"] = v[ends - cnt], v[ends - 1]
            return out
        out["avg"] = None
        if case["avg"]:
            a, = _group_sums(t["key"], g, t["avg"])
            out["avg"] = a.double() / cnt.double()
        return out
    v = torch.where(t["date"] < case["D"], t["price"] * (100 - t["disc"]), 0) + t["flag"].long()
    keep = torch.nonzero((t["date"] < case["D"]) & (v > 500_000_000)).reshape(-1)
    row = torch.zeros(case["n"], dtype=torch.int32, device="cuda")
    carried = torch.zeros(case["n"], dtype=torch.int32, device="cuda")
    row[:keep.numel()] = keep.to(torch.int32)
    carried[:keep.numel()] = t["fk"][keep]
    return {"value": v, "row": row, "carried": carried, "count": one(keep.numel())}
