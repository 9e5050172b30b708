"""Hash probes behind the table's pass filter in the fused pass (tables larger
than an XCD's L2, most rows not passing), at row counts that leave 0 to 3 rows
past the last whole item: the oracle's groups, with the filter and without."""

import numpy as np
import pytest

import datagen
from gpu_util import assert_same, oracle_rows, require_gpu, run_gpu, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("span", [900_000, 1 << 31])
def test_filtered_probe(span):
    require_gpu()
    rng = np.random.default_rng(span)
    m = 400_000                                            # 2^20 slots, 8 MB
    keys = (rng.choice(span, m, replace=False) - span // 2).astype(np.int32)
    dims = {"big": {"k": keys, "f": rng.integers(0, 4, m, dtype=np.int32), "a": rng.integers(0, 50, m, dtype=np.int32)},
            "d": {"k": np.arange(100, dtype=np.int32), "b": rng.integers(0, 7, 100, dtype=np.int32)}}
    joins = [{"fact_key": "k", "dim": "big", "preds": [{"col": "f", "op": "eq", "lo": 1, "hi": None}],
              "payloads": ["a"], "kind": "hash", "load_factor": 0.5},
             {"fact_key": "d", "dim": "d", "preds": [], "payloads": ["b"], "kind": "auto"}]
    for n in (3, 4096, 200_001, 200_002, 200_003):
        miss = rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
        fact = {"k": np.where(rng.random(n) < 0.8, keys[rng.integers(0, m, n)], miss).astype(np.int32),
                "d": rng.integers(-2, 104, n, dtype=np.int32), "v": rng.integers(-10**9, 10**9, n, dtype=np.int32)}
        w = datagen.Workload(f"{n} rows", n, fact, dims, {"big": "k", "d": "k"},
                             {"fact_preds": [], "joins": joins, "group_by": [["big", "a"], ["d", "b"]],
                              "agg": {"kind": "mul", "a": "v", "b": "k"}})
        want, dev = oracle_rows(w), upload(w)
        for force in (None, {"prefilter": -1}, {"ipt": 2}, {"terminal": "global"}, {"terminal": "part"}):
            got, _ = run_gpu(w, force=force, dev=dev)
            assert_same(got.as_rows(), want, f"{span} {n} {force}")
