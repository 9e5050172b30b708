"""The compaction of the group table in one kernel, in two, and with the scan
in between, at their edges; rank tables built in one kernel, which also zeroes
the outputs."""

from types import SimpleNamespace

import numpy as np
import pytest

import datagen
from gpu_util import assert_same, oracle_rows, require_gpu, run_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("present", ["none", "all", "some", "last"])
@pytest.mark.parametrize("groups", [1, 63, 64, 1023, 1024, 1025, 8191, 8192, 8193, 9217, 4096 * 1024, 4096 * 1024 + 1])
def test_compaction(groups, present):
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    rng = np.random.default_rng([groups, len(present)])
    counts = {"none": np.zeros(groups, np.int64), "all": rng.integers(1, 9, groups),
              "some": rng.integers(0, 3, groups), "last": np.eye(1, groups, groups - 1, dtype=np.int64)[0]}[present]
    sums = rng.integers(-(1 << 62), 1 << 62, groups)
    plan = sdb.SdbPlan()
    plan.n_group_keys, plan.n_groups = 1, groups
    plan.radix[0], plan.stride[0], plan.key_min[0] = groups, 1, -7
    q = SimpleNamespace(n_keys=1, plan_obj=plan)
    s, c = torch.from_numpy(sums).cuda(), torch.from_numpy(counts).cuda()
    k, os, oc, n, _ = sdb.StarQuery.finalize(q, s, c)
    at = np.flatnonzero(counts)
    m = int(n.item())
    assert m == at.size
    assert np.array_equal(k[:m, 0].cpu().numpy(), at - 7)
    assert np.array_equal(os[:m].cpu().numpy(), sums[at]) and np.array_equal(oc[:m].cpu().numpy(), counts[at])


def _ranked(m, groups, n=50_003):
    """A dimension of m rows, a quarter passing (the first and the last among
    them), with `groups` attribute values over the passing rows' range: 1-byte
    codes up to 254, 2-byte up to 65,534, 4-byte above."""
    rng = np.random.default_rng([m, groups])
    f, a = rng.integers(0, 4, m, dtype=np.int32), rng.integers(0, groups, m, dtype=np.int32)
    f[[0, -1]] = 1
    a[0], a[-1] = 0, groups - 1
    dims = {"d": {"k": np.arange(m, dtype=np.int32), "f": f, "a": a}}
    fact = {"k": rng.integers(-3, m + 3, n, dtype=np.int32), "v": rng.integers(-10**9, 10**9, n, dtype=np.int32)}
    query = {"fact_preds": [], "joins": [{"fact_key": "k", "dim": "d", "preds": [{"col": "f", "op": "eq", "lo": 1,
                                                                                  "hi": None}],
                                          "payloads": ["a"], "kind": "auto"}],
             "group_by": [["d", "a"]], "agg": {"kind": "col", "a": "v", "b": None}}
    return datagen.Workload(f"{m} rows, {groups} groups", n, fact, dims, {"d": "k"}, query)


@pytest.mark.parametrize("m,groups", [(8193, 70_000), (16_383, 70_000), (16_384, 70_000), (16_385, 70_000),
                                      (24_640, 70_000), (65_536, 70_000), (80_001, 70_000), (32_769, 200),
                                      (16_449, 300), (100_001, 300)])
def test_rank_tables(m, groups):
    """Dimensions past the whole map's budget as LDS rank tables, at row counts
    around the kernel's blocks (8,192 slots) and 64-slot groups."""
    w = _ranked(m, groups)
    want = oracle_rows(w)
    for force in ({"lds": 3}, {"lds": 3, "terminal": "global", "xcd": 1}, {"lds": 3, "terminal": "part"}):
        got, q = run_gpu(w, force=force)
        assert q.plan_obj.stage_lds[0] == 3
        assert_same(got.as_rows(), want, f"{w.name} {force}")


@pytest.mark.parametrize("m", [1, 31, 32, 33, 63, 64, 65, 8191, 8192, 8193])
@pytest.mark.parametrize("groups", [200, 300, 70_000])
def test_rank_tables_of_one_word_and_one_block(m, groups):
    """The smallest tables, which the planner stages whole, in a plan that asks
    for rank tables, with outputs and scratch that hold something else before."""
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    w = _ranked(m, groups)
    fact, dims = upload(w)
    q = sdb.StarQuery(fact, sdb.build_dims(dims, w.dim_keys, w.query), w.query,
                      {"terminal": "global", "xcd": -1, "block": 1024})
    plan, d = q.plan(), q.tables[0].handle
    assert d.width == ({200: 1, 300: 2, 70_000: 4}[groups] if m > 1 else 1)

    def up(b, to):
        return max(to, -(-b // to) * to)

    rank, codes = up(-(-d.n_slots // 64) * 4, 16), up(d.n_pass * d.width, 16)
    plan.stage_lds[0], plan.stage_defer[0] = 3, -1
    plan.lds_bytes = up(-(-d.n_slots // 32) * 4, 16) + rank + codes
    plan.run_scratch_bytes = up(rank, 256) + up(codes, 256)
    scratch = torch.full((plan.run_scratch_bytes,), 0xA5, dtype=torch.uint8, device="cuda")
    sums, counts = (t.fill_(-7) for t in q.alloc_outputs())
    q.run(sums, counts, scratch=scratch)
    k, s, c, n, _ = q.finalize(sums, counts)
    n = int(n.item())
    got = sdb.QueryResult(k[:n].to(torch.int64).cpu().numpy(), s[:n].cpu().numpy(), c[:n].cpu().numpy())
    assert_same(got.as_rows(), oracle_rows(w), w.name)
