"""4-row items on columns that are not 16-byte aligned: every terminal, one and
two items per lane, row counts around an item and a tile, columns at different
offsets, each against the oracle and against 1-row items (which plans with a hash
probe keep)."""

import numpy as np
import pytest

import datagen
from gpu_util import assert_same, oracle_rows, require_gpu, run_gpu, upload

pytestmark = pytest.mark.gpu


def _mixed_offsets(w):
    """The workload's columns as views 1, 2, 3, 1, ... elements into buffers
    that end with the column (nothing readable past its last row)."""
    import torch
    fact = {}
    for i, (name, v) in enumerate(w.fact.items()):
        off = 1 + i % 3
        buf = torch.empty(v.size + off, dtype=torch.int32, device="cuda")
        buf[off:] = torch.from_numpy(np.ascontiguousarray(v)).cuda()
        fact[name] = buf[off:]
    return fact, upload(w)[1]


@pytest.mark.parametrize("name,force", [("c1_scalar_scan", None), ("c2_join_group", None), ("c3_star3", None),
                                        ("c3_star3", {"terminal": "part"}), ("c3_star3", {"segments": 1}),
                                        ("c4_star4_zipf", None), ("c3_star3", {"ipt": 2}), ("c4_star4_zipf", {"ipt": 2}),
                                        ("c5_hash_stress", None)])
@pytest.mark.parametrize("n", [1, 3, 4, 2047, 2049, 300_007])
def test_unaligned_columns(name, force, n):
    require_gpu()
    w = datagen.make_workload(name, n_fact=n)
    want = oracle_rows(w)
    dev = _mixed_offsets(w)
    got, q = run_gpu(w, force=force, dev=dev)
    plan = q.plan_obj
    assert plan.vector == 0 and plan.unroll == 0
    assert plan.item_rows == (1 if name == "c5_hash_stress" else 4)
    assert plan.ipt == (1 if name in ("c3_star3", "c4_star4_zipf") and not (force or {}).get("ipt") else 2)
    assert_same(got.as_rows(), want, f"{name} {n} rows {force}")
    if n == 300_007:
        got, q = run_gpu(w, force={**(force or {}), "vector": -1}, dev=dev)
        assert q.plan_obj.item_rows == 1
        assert_same(got.as_rows(), want, f"{name} {n} rows {force}, 1-row items")
