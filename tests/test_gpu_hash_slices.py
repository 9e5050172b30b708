"""Hash tables built slice by slice (786,432 rows or more, with a Bloom filter 2^19): every row is found
where linear probing looks for it, the pass filter is as documented, and
duplicates and uneven hashes are met as by inserts."""

import numpy as np
import pytest

import datagen
from gpu_util import assert_same, oracle_rows, require_gpu, run_gpu, upload
from test_gpu_parity import _bloom_words, _filter_words

pytestmark = pytest.mark.gpu

K = 0x9E3779B1


def _dims(keys, seed, groups=300):
    rng = np.random.default_rng([2607, 7632, 91, seed])
    return {"key": keys, "flag": rng.integers(0, 2, keys.size, dtype=np.int32),
            "attr": rng.integers(-5, groups - 5, keys.size, dtype=np.int32)}


def _query(lf):
    return {"fact_preds": [],
            "joins": [{"fact_key": "key", "dim": "big", "preds": [{"col": "flag", "op": "eq", "lo": 1, "hi": None}],
                       "payloads": ["attr"], "kind": "hash", "load_factor": lf}],
            "group_by": [["big", "attr"]], "agg": {"kind": "col", "a": "value", "b": None}}


def _build(dim, lf, workspace_extra=True):
    import torch
    from paper_2607_07632_amd import sdb
    require_gpu()
    cols = {c: torch.from_numpy(a).cuda() for c, a in dim.items()}
    desc = sdb.dim_desc(*sdb._join_inputs({"big": cols}, {"big": "key"}, _query(lf)["joins"][0]))
    need = sdb.dim_required_bytes(desc) + (9 * dim["key"].size + (4 << 20) if workspace_extra else 0)
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    return sdb.build_dims({"big": cols}, {"big": "key"}, _query(lf), workspaces=[ws])[0]


def _slots(t):
    import torch
    n = int(t.handle.n_slots)
    off = t.handle.map - t.workspace.data_ptr()
    return t.workspace[off:off + 8 * n].view(torch.int64).cpu().numpy().view(np.uint64)


def _check_table(t, dim):
    """Every row in exactly one slot, holding its key and code, with no empty
    slot between its home and there."""
    slots = _slots(t)
    n, bits = slots.size, int(t.handle.hash_bits)
    at = np.flatnonzero(slots)
    keys = (slots[at] & np.uint64(0xFFFFFFFF)).astype(np.uint32)
    enc = (slots[at] >> np.uint64(32)).astype(np.uint32)
    assert at.size == dim["key"].size
    lo = int(dim["attr"][dim["flag"] == 1].min())
    want = np.where(dim["flag"] == 1, dim["attr"].astype(np.int64) - lo + 1, 0xFFFFFFFF).astype(np.uint32)
    order, mine = np.argsort(keys), np.argsort(dim["key"].view(np.uint32))
    assert np.array_equal(keys[order], dim["key"].view(np.uint32)[mine])
    assert np.array_equal(enc[order], want[mine])
    home = ((keys.astype(np.uint64) * np.uint64(K)) & np.uint64(0xFFFFFFFF)) >> np.uint64(32 - bits)
    dist = (at - home.astype(np.int64)) % n
    full = np.concatenate([[0], np.cumsum(np.concatenate([slots, slots]) != 0)])
    assert np.array_equal(full[home.astype(np.int64) + dist] - full[home.astype(np.int64)], dist)


def _was_sliced(t, m):
    """Whether the build wrote its records into the workspace past the required
    bytes: their middle, 9 bytes a row and 4 MiB before the end."""
    at = t.workspace.numel() - (9 * m + (4 << 20)) + (1 << 20) + 4 * m
    return bool((t.workspace[at:at + 4096] != 0xA5).any())


@pytest.mark.parametrize("m,lf,eighths,sliced", [
    ((1 << 19) - 1, 0.5, 4, False), (1 << 19, 0.5, 4, True), ((3 << 18) - 1, 0.5, 1, False), (3 << 18, 0.5, 1, True),
    (700_001, 0.9, 4, True), (1_300_003, 0.3, 4, True)])
def test_slots_and_filter(m, lf, eighths, sliced):
    """The smallest tables built by slices, and the largest that are not: half
    of the rows or one in eight in the Bloom filter."""
    rng = np.random.default_rng(m)
    keys = rng.choice(1 << 32, m, replace=False).astype(np.uint32).view(np.int32)
    dim = _dims(keys, m)
    dim["flag"] = (rng.integers(0, 8, m) < eighths).astype(np.int32)
    t = _build(dim, lf)
    assert _was_sliced(t, m) == sliced
    _check_table(t, dim)
    assert np.array_equal(_filter_words(t), _bloom_words(keys[dim["flag"] == 1], t.handle.filter_bits // 32))


def test_without_the_extra_workspace():
    keys = np.random.default_rng(1).choice(1 << 31, 800_000, replace=False).astype(np.int32)
    dim = _dims(keys, 1)
    _check_table(_build(dim, 0.5, workspace_extra=False), dim)


def test_uneven_hashes_fall_back_to_inserts():
    """All hashes in the lower three eighths: half of the slices there overfill."""
    inv = pow(K, -1, 1 << 32)
    h = np.random.default_rng(2).choice(3 << 29, 3 << 18, replace=False).astype(np.uint64)
    keys = ((h * np.uint64(inv)) & np.uint64(0xFFFFFFFF)).astype(np.uint32).view(np.int32)
    dim = _dims(keys, 2)
    t = _build(dim, 0.5)
    assert not _was_sliced(t, keys.size)      # (given up before a row was moved)
    _check_table(t, dim)
    assert np.array_equal(_filter_words(t), _bloom_words(keys[dim["flag"] == 1], t.handle.filter_bits // 32))


def test_full_slices_between_overfull_ones():
    """Slices of 4,096 slots: each odd one holds more rows than slots, each even
    one 3,000 rows in its last half, which spill, so no pass may probe a table
    that holds what the workspace held (0xA5) before the inserts."""
    rng = np.random.default_rng(8)
    per = 1 << 12
    h = []
    for q in range(0, 222, 2):
        h.append((q * per + per // 2) * 4096 + rng.choice(per // 2 * 4096, 3000, replace=False))
        h.append((q + 1) * per * 4096 + rng.choice(per * 4096, per + 50, replace=False))
    h = np.concatenate(h).astype(np.uint64)
    assert h.size >= 3 << 18 and h.size / 0.9 <= 1 << 20
    keys = ((h * np.uint64(pow(K, -1, 1 << 32))) & np.uint64(0xFFFFFFFF)).astype(np.uint32).view(np.int32)
    dim = _dims(rng.permutation(keys), 8)
    t = _build(dim, 0.9)
    assert int(t.handle.hash_bits) == 20
    _check_table(t, dim)
    assert np.array_equal(_filter_words(t), _bloom_words(dim["key"][dim["flag"] == 1], t.handle.filter_bits // 32))


def test_duplicates_are_reported():
    from paper_2607_07632_amd import sdb
    keys = np.random.default_rng(3).permutation(800_000).astype(np.int32) * 7
    keys[-1] = keys[5]
    with pytest.raises(sdb.SdbError) as e:
        _build(_dims(keys, 3), 0.5)
    assert e.value.name == "SDB_DUP_KEY"


def test_two_sliced_tables_and_a_dense_one_in_one_batch():
    rng = np.random.default_rng(4)
    a = rng.choice(1 << 31, 900_000, replace=False).astype(np.int32)
    b = rng.choice(1 << 31, 790_000, replace=False).astype(np.int32)
    n = 200_003
    fact = {"ka": a[rng.integers(0, a.size, n)], "kb": b[rng.integers(0, b.size, n)],
            "kc": rng.integers(0, 1000, n, dtype=np.int32), "v": rng.integers(-10**6, 10**6, n, dtype=np.int32)}
    dims = {"a": _dims(a, 5, 20), "b": _dims(b, 6, 30), "c": _dims(np.arange(1000, dtype=np.int32), 7, 4)}
    joins = [{"fact_key": "k" + d, "dim": d, "preds": [{"col": "flag", "op": "eq", "lo": 1, "hi": None}],
              "payloads": ["attr"], "kind": "auto"} for d in "abc"]
    w = datagen.Workload("two sliced", n, fact, dims, {d: "key" for d in "abc"},
                         {"fact_preds": [], "joins": joins, "group_by": [[d, "attr"] for d in "abc"],
                          "agg": {"kind": "col", "a": "v", "b": None}})
    got, _ = run_gpu(w, dev=upload(w))
    assert_same(got.as_rows(), oracle_rows(w), "two sliced tables")
