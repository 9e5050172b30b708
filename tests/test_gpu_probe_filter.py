"""Hash probes of the fused pass at row counts that leave 0 to 3 rows past the
last whole item: behind the table's pass filter (tables larger than an XCD's L2,
most rows not passing) and without it, rows that go through their chains
together and row by row. The oracle's groups each time."""

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


@pytest.mark.parametrize("m,lf", [(60_000, 0.5), (40_000, 0.5), (120_000, 0.9), (500_000, 0.5), (300_000, 0.5),
                                  (600_000, 0.9), (1_100_000, 0.5), (1_900_000, 0.9)])
@pytest.mark.parametrize("rows", [150_003, (1 << 20) + 2, 8_000_001])
def test_tables_of_every_size_and_load(m, lf, rows):
    """Up to 2 MiB, 4 and 8 MiB, 16 and more, from a quarter to nearly full:
    where the rows go on together and where row by row, most rows passing."""
    require_gpu()
    rng = np.random.default_rng(m)
    keys = rng.choice(1 << 32, m, replace=False).astype(np.uint32).view(np.int32)
    dims = {"big": {"k": keys, "f": rng.integers(0, 4, m, dtype=np.int32), "a": rng.integers(0, 50, m, dtype=np.int32)}}
    n = rows
    miss = rng.integers(-(1 << 31), 1 << 31, n).astype(np.int32)
    fact = {"k": np.where(rng.random(n) < 0.9, keys[rng.integers(0, m, n)], miss).astype(np.int32),
            "v": rng.integers(-10**9, 10**9, n, dtype=np.int32)}
    w = datagen.Workload(f"{m} rows", n, fact, dims, {"big": "k"},
                         {"fact_preds": [], "joins": [{"fact_key": "k", "dim": "big", "payloads": ["a"], "kind": "hash",
                                                       "preds": [{"col": "f", "op": "ge", "lo": 1, "hi": None}],
                                                       "load_factor": lf}],
                          "group_by": [["big", "a"]], "agg": {"kind": "col", "a": "v", "b": None}})
    want, dev = oracle_rows(w), upload(w)
    for force in (None, {"ipt": 2}, {"terminal": "global"}, {"slice": 1}) if rows < 1 << 20 else (None,):
        got, _ = run_gpu(w, force=force, dev=dev)
        assert_same(got.as_rows(), want, f"{m} {lf} {rows} {force}")
