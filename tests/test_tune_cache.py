"""The autotuner's cache file: which entries serve a call (no GPU needed; the
tuner itself is replaced by one that counts its calls)."""
import json
import types

import torch

import paper_2506_23058_amd as P
from paper_2506_23058_amd import ops


def _setup(monkeypatch, tmp_path):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("IXP_TUNE_CACHE", str(path))
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda dev: types.SimpleNamespace(gcnArchName="gfx950:x"))
    calls = []

    def tune(*a, **k):
        calls.append(1)
        return (512, 2, len(calls), 3), 0.5
    monkeypatch.setattr(ops, "tune_segmented", tune)
    return path, calls


def _call(n, m):
    return P.autotuned_tiling(torch.zeros(n, dtype=torch.int32), torch.zeros(m, dtype=torch.int64), P.Pred.mod_eq(2, 0))


def test_an_entry_serves_one_side_of_the_packing_rule(monkeypatch, tmp_path):
    """Two calls in one bin of n and m, their mean row at and past the longest that packs."""
    path, calls = _setup(monkeypatch, tmp_path)
    m = 2048
    first, second = _call(768 * m + m - 1, m), _call(769 * m, m)
    assert first[0] != second[0] and not first[2] and not second[2] and len(calls) == 2
    assert _call(767 * m, m) == (first[0], 0.5, True) and _call(770 * m, m) == (second[0], 0.5, True)
    assert _call(32 * 2047, 2047)[2] is False and len(json.loads(path.read_text())) == 3


def test_entries_from_before_packed_rows_are_not_used(monkeypatch, tmp_path):
    path, calls = _setup(monkeypatch, tmp_path)
    path.write_text(json.dumps({"tiling+rowsync|gfx950|torch.int32|0|torch.int32|0|n2^16|m2^11":
                                {"tiling": [256, 2, 16, 3], "ms": 0.1}}))
    tiling, _, cached = _call(32 * 2048, 2048)
    assert not cached and len(calls) == 1 and tiling != (256, 2, 16, 3)
    assert _call(32 * 2048, 2048)[2]
