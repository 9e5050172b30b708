"""The work that a user of this framework has it do, as cases for timing and for comparing results.

A case is a star query (one of six shapes) over synthetic tables on the GPU:

* ``scan``: SUM(price * disc) under two fact predicates and a date join (one row out);
* ``join``: SUM(revenue) GROUP BY (supplier nation, year) over one filtered dimension and the date;
* ``star3``: SUM(revenue) GROUP BY (customer city, supplier city, year) over three dimensions;
* ``star4``: SUM(revenue - supplycost) GROUP BY (year, brand, supplier nation) over four, with Zipf part keys;
* ``hash``: SUM(value) GROUP BY attr through one open-addressing table;
* ``hash2``: SUM(a * b) GROUP BY (city, segment) through two open-addressing tables and a fact predicate.

``call`` is how a program reaches it: ``run`` is the query over tables that are built and planned already
(the fused pass and the compaction of the groups, results left on the GPU), as a serving loop repeats it;
``step`` is a new batch: the dimension tables are rebuilt, the query is planned, run and compacted, and the
number of groups is read back. ``offset`` cuts the fact columns out of a larger buffer that many rows in, so
that they are not 16-byte aligned; ``by_date`` sorts the fact rows by date.
"""

import math

import torch

from paper_2607_07632_amd import sdb

DAYS = 2556
CHUNK = 1 << 26        # rows generated, or checked, at a time


def _case(name, query, rows, call="run", dim_rows=0, sparse=False, groups=0, offset=0, by_date=False):
    return {"name": name, "query": query, "rows": rows, "call": call, "dim_rows": dim_rows, "sparse": sparse,
            "groups": groups, "offset": offset, "by_date": by_date}


def listed():
    return [
        # a dashboard's filtered total over one recent partition: launches and latency count
        _case("scan_1m", "scan", 1_048_576),
        # the same total over a whole fact table: streaming
        _case("scan_400m", "scan", 400_000_000),
        # a report with a few hundred groups over a mid-size table
        _case("join_60m", "join", 60_000_000, dim_rows=200_000),
        # the same over a range of rows that starts anywhere: columns that are not 16-byte aligned, a ragged end
        _case("join_cut_20m", "join", 20_000_001, dim_rows=200_000, offset=1),
        # a three-dimension star over one day's rows: few rows, a large group domain
        _case("star3_3m", "star3", 3_000_017, dim_rows=3_000_000),
        # the same over the whole fact table (the headline workload)
        _case("star3_600m", "star3", 600_000_000, dim_rows=3_000_000),
        # a selective four-dimension star over skewed keys
        _case("star4_600m", "star4", 600_000_000, dim_rows=3_000_000),
        # a dimension larger than the caches, probed by the whole fact table
        _case("hash_600m", "hash", 600_000_000, dim_rows=1 << 24, groups=65_536),
        # keys of an outside system, spread over the whole int32 range, into a mid-size dimension
        _case("hash_sparse_40m", "hash", 40_000_003, dim_rows=1_500_000, sparse=True, groups=1_000),
        # two such dimensions in one query
        _case("hash2_24m", "hash2", 24_000_000, dim_rows=500_000, sparse=True, groups=250),
        # a new batch of 2M rows against freshly loaded dimensions
        _case("step_star3_2m", "star3", 2_000_000, call="step", dim_rows=3_000_000),
        # a new batch against a freshly loaded dimension of outside keys
        _case("step_hash_30m", "hash", 30_000_000, call="step", dim_rows=1 << 23, sparse=True, groups=5_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    query = rng.choice(["scan", "join", "star3", "star4", "hash", "hash2"])
    call = "step" if rng.random() < 0.25 else "run"
    offset = rng.choice([1, 2, 3]) if rng.random() < 0.2 else 0
    top = 100_000_000 if call == "step" or offset or query == "hash2" else 300_000_000
    rows = _log(rng, 100_000, top)
    case = {"query": query, "rows": rows, "call": call, "dim_rows": 0, "sparse": False, "groups": 0,
            "offset": offset, "by_date": False}
    if query == "join":
        case["dim_rows"] = _log(rng, 2_000, 1_000_000)
    elif query in ("star3", "star4"):
        case["dim_rows"] = _log(rng, 30_000, 3_000_000)
        case["by_date"] = query == "star3" and rng.random() < 0.3
    elif query == "hash":
        case["dim_rows"] = _log(rng, 50_000, 1 << 24)
        case["sparse"] = rng.random() < 0.6
        case["groups"] = _log(rng, 10, 65_536)
    elif query == "hash2":
        case["dim_rows"] = _log(rng, 20_000, 2_000_000)
        case["sparse"] = True
        case["groups"] = _log(rng, 5, 500)
    return case


# ---- tables and queries -------------------------------------------------------------------------------------

def _pred(col, op, lo, hi=None):
    return {"col": col, "op": op, "lo": lo, "hi": hi}


def _query(case):
    date_years = {"fact_key": "date_key", "dim": "date", "preds": [_pred("year", "between", 1992, 1997)],
                  "payloads": ["year"], "kind": "auto"}
    region = [_pred("region", "eq", 2)]
    if case["query"] == "scan":
        return {"fact_preds": [_pred("disc", "between", 2, 4), _pred("qty", "lt", 30)],
                "joins": [{"fact_key": "date_key", "dim": "date", "preds": [_pred("year", "eq", 1994)],
                           "payloads": [], "kind": "auto"}],
                "group_by": [], "agg": {"kind": "mul", "a": "price", "b": "disc"}}
    if case["query"] == "join":
        return {"fact_preds": [],
                "joins": [{"fact_key": "supp_key", "dim": "supplier", "preds": region, "payloads": ["nation"],
                           "kind": "auto"},
                          {"fact_key": "date_key", "dim": "date", "preds": [], "payloads": ["year"], "kind": "auto"}],
                "group_by": [["supplier", "nation"], ["date", "year"]], "agg": {"kind": "col", "a": "revenue", "b": None}}
    if case["query"] == "star3":
        return {"fact_preds": [],
                "joins": [{"fact_key": "cust_key", "dim": "customer", "preds": region, "payloads": ["city"],
                           "kind": "auto"},
                          {"fact_key": "supp_key", "dim": "supplier", "preds": region, "payloads": ["city"],
                           "kind": "auto"}, date_years],
                "group_by": [["customer", "city"], ["supplier", "city"], ["date", "year"]],
                "agg": {"kind": "col", "a": "revenue", "b": None}}
    if case["query"] == "star4":
        return {"fact_preds": [],
                "joins": [{"fact_key": "part_key", "dim": "part", "preds": [_pred("category", "eq", 1)],
                           "payloads": ["brand"], "kind": "auto"},
                          {"fact_key": "cust_key", "dim": "customer", "preds": region, "payloads": [], "kind": "auto"},
                          {"fact_key": "supp_key", "dim": "supplier", "preds": region, "payloads": ["nation"],
                           "kind": "auto"}, date_years],
                "group_by": [["date", "year"], ["part", "brand"], ["supplier", "nation"]],
                "agg": {"kind": "sub", "a": "revenue", "b": "supplycost"}}
    if case["query"] == "hash":
        return {"fact_preds": [],
                "joins": [{"fact_key": "key", "dim": "big", "preds": [_pred("flag", "eq", 1)], "payloads": ["attr"],
                           "kind": "hash", "load_factor": 0.5}],
                "group_by": [["big", "attr"]], "agg": {"kind": "col", "a": "value", "b": None}}
    return {"fact_preds": [_pred("qty", "lt", 40)],
            "joins": [{"fact_key": "acct_key", "dim": "account", "preds": [_pred("flag", "eq", 1)],
                       "payloads": ["city"], "kind": "auto"},
                      {"fact_key": "item_key", "dim": "item", "preds": [], "payloads": ["segment"], "kind": "auto"}],
            "group_by": [["account", "city"], ["item", "segment"]], "agg": {"kind": "mul", "a": "price", "b": "qty"}}


class _Maker:
    """int32 columns on the GPU from one seeded generator."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def uniform(self, n, lo, hi, out=None):
        """n whole values lo .. hi."""
        if out is None:
            out = torch.empty(n, dtype=torch.int32, device="cuda")
        return out.random_(int(lo), int(hi) + 1, generator=self.g)

    def zipf(self, out, n_keys, s):
        """Ranks 0 .. n_keys - 1 with P(rank r) proportional to (r + 1) ** -s."""
        cdf = torch.arange(1, n_keys + 1, dtype=torch.float64, device="cuda").pow_(-s).cumsum_(0)
        cdf /= cdf[-1].clone()
        for a in range(0, out.numel(), CHUNK):
            b = min(out.numel(), a + CHUNK)
            u = torch.rand(b - a, dtype=torch.float64, device="cuda", generator=self.g)
            out[a:b] = torch.searchsorted(cdf, u, right=True).clamp_(max=n_keys - 1)

    def keys(self, n, sparse):
        """n distinct keys in random order: 0 .. n - 1, or spread over the non-negative int32 range."""
        order = torch.randperm(n, device="cuda", generator=self.g)
        if not sparse:
            return order.to(torch.int32)
        gap = (1 << 31) // n
        return (order * gap + self.uniform(n, 0, gap - 1)).to(torch.int32)

    def picks(self, out, keys, sparse):
        """Fact keys: uniform over the dimension's keys; with spread keys one in eight is in no dimension row
        (but for chance)."""
        for a in range(0, out.numel(), CHUNK):
            b = min(out.numel(), a + CHUNK)
            at = self.uniform(b - a, 0, keys.numel() - 1)
            v = keys[at.long()]
            if sparse:
                v = torch.where(self.uniform(b - a, 0, 7) == 0, self.uniform(b - a, 0, (1 << 31) - 2), v)
            out[a:b] = v


def _date():
    d = torch.arange(DAYS, device="cuda")
    return {"date_key": d.to(torch.int32), "year": (1992 + torch.div(d, 365, rounding_mode="floor")).to(torch.int32)}


def _index(n):
    return torch.arange(n, dtype=torch.int32, device="cuda")


def _tables(case, seed):
    """(fact columns, dimension tables, their key columns)."""
    m = _Maker(seed)
    n, d, off = case["rows"], case["dim_rows"], case["offset"]

    def column():
        return torch.empty(n + 4, dtype=torch.int32, device="cuda")[off:off + n] if off else \
            torch.empty(n, dtype=torch.int32, device="cuda")

    fact, dims = {}, {}

    def uniform(name, lo, hi):
        fact[name] = m.uniform(n, lo, hi, column())

    def date_key():
        if not case["by_date"]:
            return uniform("date_key", 0, DAYS - 1)
        out = column()
        for a in range(0, n, CHUNK):
            b = min(n, a + CHUNK)
            out[a:b] = torch.div(torch.arange(a, b, device="cuda") * DAYS, n, rounding_mode="floor")
        fact["date_key"] = out

    if case["query"] == "scan":
        date_key()
        uniform("qty", 1, 50)
        uniform("disc", 0, 10)
        uniform("price", 90_000, 10_000_000)
        dims["date"] = _date()
    elif case["query"] == "join":
        uniform("supp_key", 0, d - 1)
        date_key()
        uniform("revenue", 1, 1_000_000)
        dims["supplier"] = {"supp_key": _index(d), "region": m.uniform(d, 0, 4), "nation": m.uniform(d, 0, 24)}
        dims["date"] = _date()
    elif case["query"] in ("star3", "star4"):
        supp, part = max(2_000, d // 15), max(2_000, d * 7 // 15)
        uniform("cust_key", 0, d - 1)
        uniform("supp_key", 0, supp - 1)
        date_key()
        uniform("revenue", 1, 1_000_000)
        dims["customer"] = {"cust_key": _index(d), "region": m.uniform(d, 0, 4), "city": m.uniform(d, 0, 249)}
        dims["supplier"] = {"supp_key": _index(supp), "region": m.uniform(supp, 0, 4),
                            "city": m.uniform(supp, 0, 249), "nation": m.uniform(supp, 0, 24)}
        dims["date"] = _date()
        if case["query"] == "star4":
            uniform("supplycost", 1, 100_000)
            fact["part_key"] = column()
            m.zipf(fact["part_key"], part, 1.1)
            dims["part"] = {"part_key": _index(part), "category": m.uniform(part, 0, 24), "brand": m.uniform(part, 0, 999)}
    elif case["query"] == "hash":
        dims["big"] = {"key": m.keys(d, case["sparse"]), "flag": m.uniform(d, 0, 1),
                       "attr": m.uniform(d, 0, case["groups"] - 1)}
        fact["key"] = column()
        m.picks(fact["key"], dims["big"]["key"], case["sparse"])
        uniform("value", 1, 1_000_000)
    else:
        items = max(1_000, d // 10)
        dims["account"] = {"acct_key": m.keys(d, True), "flag": m.uniform(d, 0, 2),
                           "city": m.uniform(d, 0, case["groups"] - 1)}
        dims["item"] = {"item_key": m.keys(items, True), "segment": m.uniform(items, 0, 6)}
        for name, dim in (("acct_key", "account"), ("item_key", "item")):
            fact[name] = column()
            m.picks(fact[name], dims[dim][name], True)
        uniform("qty", 1, 50)
        uniform("price", 1, 1_000_000)
    # every attribute's first and last value is held by a passing row: the group domain is the attributes' own, as in
    # large tables, and the result has the same shape for every seed (the last rows: the rarest of the Zipf parts)
    ends = {"nation": 24, "city": case["groups"] - 1 if case["query"] == "hash2" else 249, "brand": 999,
            "attr": case["groups"] - 1, "segment": 6}
    passing = {"region": 2, "category": 1, "flag": 1}
    for t in dims.values():
        for name, v in t.items():
            if name in passing:
                v[-2:] = passing[name]
            elif name in ends:
                v[-2] = 0
                v[-1] = ends[name]
    keys = {"date": "date_key", "supplier": "supp_key", "customer": "cust_key", "part": "part_key", "big": "key",
            "account": "acct_key", "item": "item_key"}
    return fact, dims, keys


# ---- one pass -----------------------------------------------------------------------------------------------

def prepare(case, seed):
    fact, dims, keys = _tables(case, seed)
    query = _query(case)
    prepared = sdb.PreparedDims(dims, keys, query)
    state = {"case": case, "prepared": prepared, "dims": dims}
    state["q"] = q = sdb.StarQuery(fact, prepared.tables, query)
    # tables and plan in hand, outputs and scratch allocated once
    prepared.build()
    plan = q.plan()
    q.run_scratch()
    state["sums"], state["counts"] = q.alloc_outputs()
    state["out"] = q.finalize(state["sums"].zero_(), state["counts"].zero_())
    for t in state["out"]:
        t.zero_()
    assert int(plan.n_groups) == state["sums"].numel()
    return state


def run(state):
    q, step = state["q"], state["case"]["call"] == "step"
    if step:
        state["prepared"].build()
        q.plan()
    q.run(state["sums"], state["counts"])
    keys, sums, counts, n, _ = q.finalize(state["sums"], state["counts"], outputs=state["out"])
    return {"n": int(n.item()) if step else n, "keys": keys, "sums": sums, "counts": counts}


# ---- what a pass cannot do without, and what it must give ----------------------------------------------------

def _lines(f):
    """Share of 128-byte lines of an int32 column that hold a row of a share f of the rows."""
    return 1.0 - (1.0 - f) ** 32


def work(case):
    n, d = case["rows"], case["dim_rows"]
    # the share of the rows that is left where each column is first needed, the most selective filter first
    year, hits = 6 * 365 / DAYS, 7 / 8 if case["sparse"] else 1.0
    live = {"scan": [1.0, 365 / DAYS, 365 / DAYS * 3 / 11, 365 / DAYS * 3 / 11 * 29 / 50], "join": [1.0, 0.2, 0.2],
            "star3": [1.0, 0.2, 0.04, 0.04 * year],
            # the share of the Zipf rows whose part passes varies with the draw: its mean
            "star4": [1.0, 0.04, 0.008, 0.0016, 0.0016 * year, 0.0016 * year],
            "hash": [1.0, hits / 2], "hash2": [1.0, hits / 3, hits * hits / 3, hits * hits / 3 * 39 / 50]}[case["query"]]
    total = 4.0 * n * sum(_lines(f) for f in live)
    cols = {"scan": [(DAYS, 2)], "join": [(d, 3), (DAYS, 2)], "star3": [(d, 3), (max(2_000, d // 15), 3), (DAYS, 2)],
            "star4": [(d, 2), (max(2_000, d // 15), 3), (max(2_000, d * 7 // 15), 3), (DAYS, 2)], "hash": [(d, 3)],
            "hash2": [(d, 3), (max(1_000, d // 10), 2)]}[case["query"]]
    # a dense table's code is a byte or two a row, an open-addressing table's entry 8 bytes; a step reads the columns
    per_row = 8 if case["sparse"] or case["query"] == "hash" else 1
    total += sum(r * (4 * c if case["call"] == "step" else per_row) for r, c in cols)
    groups = {"scan": 1, "join": 200, "star3": 250 * 250 * 6, "star4": 6 * 1000 * 25, "hash": case["groups"],
              "hash2": 7 * case["groups"]}[case["query"]]
    keys = {"scan": 0, "join": 2, "star3": 3, "star4": 3, "hash": 1, "hash2": 2}[case["query"]]
    total += min(groups, max(1, n * live[-1])) * (16 + 4 * keys)
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"     # sums modulo 2^64 and counts


def _holds(p, x):
    x = x.long()
    return {"eq": lambda: x == p["lo"], "lt": lambda: x < p["lo"],
            "between": lambda: (x >= p["lo"]) & (x <= p["hi"])}[p["op"]]()


def exact(case, seed):
    """The query by its definition in plain torch: every fact key looked up in the sorted dimension keys."""
    fact, dims, keys = _tables(case, seed)
    query = _query(case)
    looked, codes = [], {}
    for jd in query["joins"]:
        t = dims[jd["dim"]]
        order = torch.argsort(t[keys[jd["dim"]]])
        ok = torch.ones(order.numel(), dtype=torch.bool, device="cuda")
        for p in jd["preds"]:
            ok &= _holds(p, t[p["col"]])
        for name in jd["payloads"]:
            seen = t[name][ok].long()
            lo = int(seen.min()) if seen.numel() else 0
            codes[jd["dim"], name] = (lo, (int(seen.max()) if seen.numel() else 0) - lo + 1)
        looked.append((t[keys[jd["dim"]]][order], ok[order], order))
    shape = [codes[tuple(k)] for k in query["group_by"]]
    groups = math.prod(r for _, r in shape)
    sums = torch.zeros(groups, dtype=torch.int64, device="cuda")
    counts = torch.zeros_like(sums)
    step = CHUNK // 2
    for a in range(0, case["rows"], step):
        part = {c: x[a:a + step] for c, x in fact.items()}
        live = torch.ones(next(iter(part.values())).numel(), dtype=torch.bool, device="cuda")
        for p in query["fact_preds"]:
            live &= _holds(p, part[p["col"]])
        at = {}
        for jd, (ks, ok, order) in zip(query["joins"], looked):
            i = torch.searchsorted(ks, part[jd["fact_key"]]).clamp_(max=ks.numel() - 1)
            live &= (ks[i] == part[jd["fact_key"]]) & ok[i]
            at[jd["dim"]] = (i, order)
        group = torch.zeros(int(live.sum()), dtype=torch.int64, device="cuda")
        for (dim, name), (lo, radix) in zip(query["group_by"], shape):
            i, order = at[dim]
            group = group * radix + dims[dim][name][order[i[live]]].long() - lo
        v = part[query["agg"]["a"]][live].long()
        if query["agg"]["kind"] == "mul":
            v = v * part[query["agg"]["b"]][live].long()
        elif query["agg"]["kind"] == "sub":
            v = v - part[query["agg"]["b"]][live].long()
        sums.index_add_(0, group, v)
        counts.index_add_(0, group, torch.ones_like(group))
    found = torch.nonzero(counts).flatten() if shape else torch.zeros(1, dtype=torch.int64, device="cuda")
    out_keys = torch.zeros(groups, max(len(shape), 1), dtype=torch.int32, device="cuda")
    rest = found
    for k in range(len(shape) - 1, -1, -1):
        lo, radix = shape[k]
        out_keys[:found.numel(), k] = (rest % radix + lo).to(torch.int32)
        rest = torch.div(rest, radix, rounding_mode="floor")
    out_sums, out_counts = torch.zeros_like(sums), torch.zeros_like(counts)
    out_sums[:found.numel()], out_counts[:found.numel()] = sums[found], counts[found]
    n = found.numel()
    return {"n": n if case["call"] == "step" else torch.tensor([n], dtype=torch.int64, device="cuda"), "keys": out_keys,
            "sums": out_sums, "counts": out_counts}
