"""The sliced hash probe's LDS route (rows partitioned by table slice, summed
by dimension row in LDS) where it can go wrong: slices that overfill the LDS
table, runs past a slice's end and around the table's, hot keys split over
work items, every way the groups leave, a scratch that only holds the route
through L2, and that route. Everything is compared with the oracle, exactly."""

import numpy as np
import pytest

import datagen
from gpu_util import assert_same, oracle_rows, require_gpu, upload

pytestmark = pytest.mark.gpu

INV = pow(0x9E3779B1, -1, 1 << 32)      # the hash is key * 0x9E3779B1 mod 2^32


def _keys_of_hashes(h):
    return ((np.asarray(h, dtype=np.uint64) * INV) & 0xFFFFFFFF).astype(np.uint32).view(np.int32)


def _workload(keys, n, seed, attr=None, groups=700, lf=0.5, fact_key=None, preds=True, agg="col"):
    rng = np.random.default_rng([2607, 7632, 81, seed])
    m = keys.size
    if attr is None:
        attr = rng.integers(0, groups, m, dtype=np.int32)
    flag = rng.integers(0, 2, m, dtype=np.int32) if preds else np.ones(m, np.int32)
    hit = keys[rng.integers(0, m, n)]
    miss = rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    fact = {"key": np.where(rng.random(n) < 0.8, hit, miss).astype(np.int32) if fact_key is None else fact_key,
            "value": rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32),
            "other": rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)}
    query = {"fact_preds": [{"col": "other", "op": "ge", "lo": -2_000_000_000, "hi": None}],
             "joins": [{"fact_key": "key", "dim": "big", "preds": [{"col": "flag", "op": "eq", "lo": 1, "hi": None}],
                        "payloads": ["attr"] if groups else [], "kind": "hash", "load_factor": lf}],
             "group_by": [["big", "attr"]] if groups else [],
             "agg": {"kind": agg, "a": "value", "b": None if agg == "col" else "other"}}
    return datagen.Workload(f"seed {seed}", n, fact, {"big": {"key": keys, "flag": flag, "attr": attr}},
                            {"big": "key"}, query)


def _lds_bits(d):
    """The slices the planner gives a table of this many passing rows."""
    return next(b for b in range(8, 12) if (d.n_pass >> b) <= 4096 or b == 11)


def _check(w, force=None, label="", through_l2=False, bits=None):
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    fact, dims = upload(w)
    q = sdb.StarQuery(fact, sdb.build_dims(dims, w.dim_keys, w.query), w.query, {"slice": 1, **(force or {})})
    plan = q.plan()
    # (so few rows run through L2 unless the plan says otherwise)
    assert plan.slice_bits > 0 and plan.slice_lds == 0
    if not through_l2:
        d = q.tables[0].handle
        plan.slice_lds = min(bits or _lds_bits(d), d.hash_bits)
    sums, counts = q.alloc_outputs()
    # (a plan for so few rows does not count the LDS route's scratch)
    need = int(plan.run_scratch_bytes) + (0 if through_l2 else 128 << 20)
    scratch = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    q.run(sums, counts, scratch=scratch)
    k, s, c, n, _ = q.finalize(sums, counts)
    m = int(n.item())
    got = sdb.QueryResult(k[:m, :q.n_keys].to(torch.int64).cpu().numpy().reshape(m, q.n_keys), s[:m].cpu().numpy(),
                          c[:m].cpu().numpy())
    assert_same(got.as_rows(), oracle_rows(w), f"{w.name} {force} {label}")


@pytest.mark.parametrize("first", [0, (1 << 32) - (6000 << 10)])
def test_a_slice_that_overfills_the_table(first):
    """6,000 keys whose hashes lie in one slice (the first, or the last, whose
    run of slots wraps around the table's end): more than the LDS table's
    4,608 entries, in runs far past the slice's end."""
    keys = _keys_of_hashes(first + (np.arange(6000, dtype=np.uint64) << 10))
    for agg in ("col", "mul"):
        _check(_workload(keys, 70_001, 1, lf=0.25, preds=False, agg=agg), label=agg)
    _check(_workload(keys, 70_001, 2, lf=0.9), label="half pass")


def test_slices_of_more_than_65536_slots():
    keys = np.random.default_rng(5).choice(1 << 31, 2000, replace=False).astype(np.int32)
    _check(_workload(keys, 30_003, 3, lf=0.0001))


@pytest.mark.parametrize("groups,force", [(0, None), (1, None), (1024, None), (1025, None), (5000, None),
                                          (5000, {"terminal": "part"}), (70_000, None), (1_100_000, None),
                                          (5000, {"terminal": "global", "xcd": 1}), (300, {"terminal": "global", "xcd": 1}),
                                          (300, {"terminal": "global", "xcd": -1})])
def test_every_way_the_groups_leave(groups, force):
    """Scalar and few groups (a block's LDS), more (records by range of 4,096
    groups), more than 256 ranges (atomics), per-XCD copies."""
    keys = np.random.default_rng(6).choice(1 << 31, 40_000, replace=False).astype(np.int32)
    attr = np.random.default_rng(7).integers(0, max(groups, 1), keys.size, dtype=np.int32)
    attr[:2] = 0, max(groups, 1) - 1
    w = _workload(keys, 200_003, 8, attr=attr, groups=groups)
    w.dims["big"]["flag"][:2] = 1
    _check(w, force)


def test_records_past_a_ranges_capacity():
    """All rows but one in the first of 25 ranges of groups."""
    keys = np.random.default_rng(9).choice(1 << 31, 60_000, replace=False).astype(np.int32)
    attr = np.random.default_rng(10).integers(0, 4096, keys.size, dtype=np.int32)
    attr[0] = 100_000
    w = _workload(keys, 300_007, 11, attr=attr, preds=False)
    _check(w)


@pytest.mark.parametrize("share", [0.3, 0.6, 1.0])
@pytest.mark.parametrize("groups,agg", [(700, "col"), (5000, "mul"), (5000, "col")])
def test_hot_keys_among_others(share, groups, agg):
    """Rows that a wave adds up itself beside others of its slice, misses and
    rows that do not pass, over many work items of two slices; two hot keys,
    the int32 extremes among their values."""
    rng = np.random.default_rng(18)
    keys = rng.choice(1 << 31, 40_000, replace=False).astype(np.int32)
    n = 300_007
    w = _workload(keys, n, 18, groups=groups, agg=agg)
    w.dims["big"]["flag"][:3] = 1, 1, 0
    hot = keys[np.minimum(rng.integers(0, 6, n), 2)[:n]]        # the third is filtered out
    w.fact["key"][:] = np.where(rng.random(n) < share, hot, w.fact["key"])
    w.fact["value"][:64] = -(1 << 31)
    w.fact["other"][64:128] = (1 << 31) - 1
    _check(w)


def test_a_hot_key_over_several_work_items():
    """1.2M rows of one key (many work items of one partition), the int32
    extremes among their values."""
    keys = np.arange(-500, 500, dtype=np.int32)
    n = 1_200_003
    fk = np.full(n, 77, np.int32)
    fk[::1000] = np.arange(fk[::1000].size, dtype=np.int32) - 600
    w = _workload(keys, n, 12, fact_key=fk, preds=False)
    w.fact["value"][:3] = -(1 << 31), (1 << 31) - 1, -(1 << 31)
    _check(w)


@pytest.mark.parametrize("n", [1, 5, 4099, 16_384, 131_075])
def test_both_routes_at_chunk_edges(n):
    """The LDS route, and the route through L2, which a plan for so few rows takes."""
    keys = np.random.default_rng(13).choice(1 << 31, 3000, replace=False).astype(np.int32)
    w = _workload(keys, n, 14, groups=5000)
    for agg in ("col", "sub"):
        w.query["agg"] = {"kind": agg, "a": "value", "b": None if agg == "col" else "other"}
        for l2 in (False, True):
            _check(w, {"terminal": "global", "xcd": -1}, f"{agg}, {'L2' if l2 else 'LDS'}", l2)


def test_the_planners_route_and_a_scratch_that_holds_the_other_alone():
    """2^24 rows and a table of 2^21 slots: slices summed in LDS; with the
    pre-filter forced, a plan for the run through L2; and a plan for LDS whose
    scratch is short of it, but not of the run through L2 that it describes too."""
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    rng = np.random.default_rng(15)
    keys = rng.permutation(1 << 20).astype(np.int32)
    w = _workload(keys, 1 << 24, 15, groups=900)
    want = oracle_rows(w)
    fact, dims = upload(w)
    tables = sdb.build_dims(dims, w.dim_keys, w.query)
    for force, lds, short in (
            (None, 8, 0), ({"prefilter": 1}, 0, 0), ({"prefilter": -1}, 8, 0), ({"prefilter": -1}, 8, 65_536)):
        q = sdb.StarQuery(fact, tables, w.query, force)
        plan = q.plan()
        assert plan.slice_bits > 0 and plan.slice_lds == lds
        st = sdb.plan_summary(plan, w.query)["stages"][plan.slice_stage]
        assert st["slices_in"] == ("lds" if lds else "l2") and st["table_slices"] == 1 << (lds or plan.slice_bits)
        sums, counts = q.alloc_outputs()
        scratch = torch.full((int(plan.run_scratch_bytes) - short,), 0xA5, dtype=torch.uint8, device="cuda")
        q.run(sums, counts, scratch=scratch)
        k, s, c, n, _ = q.finalize(sums, counts)
        m = int(n.item())
        got = sdb.QueryResult(k[:m].to(torch.int64).cpu().numpy(), s[:m].cpu().numpy(), c[:m].cpu().numpy())
        assert_same(got.as_rows(), want, f"{force} {lds} {short}")


def test_the_route_in_a_graph():
    """Captured with the compaction and replayed three times, outputs and scratch
    scribbled over and other work done in between."""
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    keys = np.random.default_rng(17).choice(1 << 31, 30_000, replace=False).astype(np.int32)
    w = _workload(keys, 150_001, 17, groups=5000)
    want = oracle_rows(w)
    fact, dims = upload(w)
    q = sdb.StarQuery(fact, sdb.build_dims(dims, w.dim_keys, w.query), w.query, {"slice": 1})
    plan = q.plan()
    plan.slice_lds = 8
    scratch = torch.empty(int(plan.run_scratch_bytes) + (64 << 20), dtype=torch.uint8, device="cuda")
    sums, counts = q.alloc_outputs()
    q.run(sums, counts, scratch=scratch)
    out = q.finalize(sums, counts)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        q.run(sums, counts, scratch=scratch)
        q.finalize(sums, counts, outputs=out)
    for i in range(3):
        for t in (sums, counts, scratch, *out):
            t.fill_(0x5A + i)
        (fact["value"].sum() + i).item()
        graph.replay()
        torch.cuda.synchronize()
        k, s, c, n, _ = out
        m = int(n.item())
        got = sdb.QueryResult(k[:m].to(torch.int64).cpu().numpy(), s[:m].cpu().numpy(), c[:m].cpu().numpy())
        assert_same(got.as_rows(), want, f"replay {i}")


@pytest.mark.parametrize("agg,lds", [("col", 9), ("sub", 9)])
def test_a_large_table_few_of_whose_rows_pass(agg, lds):
    """2^23 dimension rows in 2^24 slots, a tenth passing: 512 slices of 2^15
    slots, whose runs' slot numbers stay below 2^16 (256 slices would hold the
    passing rows, but not the slots)."""
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    rng = np.random.default_rng(16)
    keys = rng.permutation(1 << 23).astype(np.int32)
    w = _workload(keys, (1 << 24) + 3, 16, groups=3000, agg=agg)
    w.dims["big"]["flag"][:] = rng.integers(0, 10, keys.size) == 1
    fact, dims = upload(w)
    q = sdb.StarQuery(fact, sdb.build_dims(dims, w.dim_keys, w.query), w.query)
    plan = q.plan()
    assert plan.slice_lds == lds and q.tables[0].handle.hash_bits == 24
    assert_same(q.execute().as_rows(), oracle_rows(w), agg)
    if agg == "col":     # and in several rounds a slice, which a plan may still ask for
        plan = q.plan_obj
        plan.slice_lds = 8
        sums, counts = q.alloc_outputs()
        q.run(sums, counts, scratch=torch.empty(int(plan.run_scratch_bytes) + (64 << 20), dtype=torch.uint8, device="cuda"))
        again = q.alloc_outputs()
        plan.slice_lds = lds
        q.run(*again)
        assert bool((sums == again[0]).all()) and bool((counts == again[1]).all())
        # so few rows past the predicate do not pay for reading the whole table: through L2
        w.query["fact_preds"][0]["lo"] = 2_080_000_000
        few = sdb.StarQuery(fact, q.tables, w.query)
        assert few.plan().slice_lds == 0 and few.plan_obj.slice_bits > 0
        assert_same(few.execute().as_rows(), oracle_rows(w), "few rows")
