"""The compaction of the group table in one kernel, in two, and with the scan
in between, at their edges; rank tables built in one kernel, which also zeroes
the outputs."""

from types import SimpleNamespace

import numpy as np
import pytest

import datagen
from gpu_util import assert_same, oracle_rows, require_gpu, run_gpu

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


@pytest.mark.parametrize("m", [1, 31, 33, 64, 8191, 8192, 8193, 100_001, 262_144])
def test_rank_tables(m):
    """A dimension of m rows (half pass) as LDS rank tables, all but the
    smallest forced past the whole map by its size."""
    rng = np.random.default_rng(m)
    dims = {"d": {"k": np.arange(m, dtype=np.int32), "f": rng.integers(0, 4, m, dtype=np.int32),
                  "a": rng.integers(0, 300, m, dtype=np.int32)}}
    n = 50_003
    fact = {"k": rng.integers(-3, m + 3, n, dtype=np.int32), "v": rng.integers(-10**9, 10**9, n, dtype=np.int32)}
    query = {"fact_preds": [], "joins": [{"fact_key": "k", "dim": "d", "preds": [{"col": "f", "op": "eq", "lo": 1,
                                                                                  "hi": None}],
                                          "payloads": ["a"], "kind": "auto"}],
             "group_by": [["d", "a"]], "agg": {"kind": "col", "a": "v", "b": None}}
    w = datagen.Workload(f"{m} rows", n, fact, dims, {"d": "k"}, query)
    for force in ({"lds": 3}, {"lds": 3, "terminal": "global", "xcd": 1}, {"lds": 3, "terminal": "part"}):
        got, q = run_gpu(w, force=force)
        # (the rank tables of 262,144 rows do not fit, smaller maps are staged whole)
        assert m != 100_001 or q.plan_obj.stage_lds[0] == 3
        assert_same(got.as_rows(), oracle_rows(w), f"{m} rows {force}")
