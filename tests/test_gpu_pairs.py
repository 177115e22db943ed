"""get_smallest_pairs (Section 6, maximal matching) on the GPU, bit-exact
against the CPU oracle; the outputs pass the device Inj checker."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

import paper_2506_23058_amd as P  # noqa: E402

DEV = "cuda:0"


def _run(n_verts, n_es, es, is_):
    print(f"[pairs] n_verts={n_verts} m={len(es)}", flush=True)
    eo, io = P.get_smallest_pairs(n_verts, n_es, torch.from_numpy(es).to(DEV), torch.from_numpy(is_).to(DEV))
    re, ri = O.get_smallest_pairs(n_verts, n_es, es, is_)
    assert np.array_equal(eo.cpu().numpy(), re) and np.array_equal(io.cpu().numpy(), ri)
    return eo, io


@pytest.mark.parametrize("n_verts,m", [(1, 1), (1, 1000), (7, 5), (1000, 3), (5000, 100_003),
                                       (1 << 20, 1 << 22)])
def test_pairs_match_oracle(n_verts, m):
    g = np.random.default_rng(n_verts * 7 + m)
    es = g.integers(0, n_verts, m)
    is_ = g.permutation(2 * m)[:m]
    eo, io = _run(n_verts, 2 * m, es, is_)
    v = P.verdicts(P.check_props(eo, P.INJ, lo=0, hi=n_verts))
    assert v[2][0] == 1   # Inj is bit 2
    v = P.verdicts(P.check_props(io, P.INJ, lo=0, hi=2 * m))
    assert v[2][0] == 1   # Inj is bit 2


def test_pairs_edge_cases():
    _run(4, 10, np.zeros(0, np.int64), np.zeros(0, np.int64))
    _run(0, 10, np.array([0, 1], np.int64), np.array([3, 4], np.int64))   # no vertices: nothing kept
    _run(3, 10, np.array([5, -1, 2, 2, 9], np.int64), np.array([0, 1, 7, 2, 3], np.int64))
    g = np.random.default_rng(5)
    es = np.where(g.random(10_001) < 0.1, -3, g.integers(0, 100, 10_001))   # out-of-range endpoints
    _run(100, 20_002, es, g.permutation(20_002)[:10_001])


def _fused(n_verts, n_es, es, is_):
    sp = P.SmallestPairs(n_verts, n_es, torch.from_numpy(es).to(DEV), torch.from_numpy(is_).to(DEV))
    assert sp.fused
    for _ in range(2):   # the second call finds the buffers of the first
        eo, io = sp()
        re, ri = O.get_smallest_pairs(n_verts, n_es, es, is_)
        assert np.array_equal(eo.cpu().numpy(), re) and np.array_equal(io.cpu().numpy(), ri)
    assert np.array_equal(sp.hist.cpu().numpy(), O.hist_min(n_verts, n_es, es, is_))


@pytest.mark.parametrize("n_verts", [1, 2047, 2049, 5000, 1 << 20, (1 << 24) - 1, (1 << 24) + 1, 1 << 25])
@pytest.mark.parametrize("m", [1, 5, 16383, 16384, 16385, 70_000])
def test_fused_pairs_match_oracle(n_verts, m, monkeypatch):
    """The fused call at the edges of its chunks (16384 entries) and bucket
    widths (1 to 2^14 vertices): uniform endpoints, runs of one bucket longer than 16
    and than 256 entries, endpoints out of range, equal ids, ids beyond the
    neutral element and negative ones."""
    monkeypatch.setattr(P.SmallestPairs, "FUSED_MIN", 0)
    g = np.random.default_rng(n_verts + m)
    es = g.integers(0, n_verts, m)
    _fused(n_verts, m, es, g.permutation(m))
    _fused(n_verts, m, np.where(g.random(m) < 0.5, n_verts - 1, es), g.integers(-9, m + 9, m))
    _fused(n_verts, m // 2, np.where(g.random(m) < 0.2, g.integers(-3, 2 * n_verts + 3, m), es),
           g.integers(0, m // 4 + 1, m))


def test_fused_pairs_large():
    g = np.random.default_rng(3)
    m = (1 << 21) + 12_345
    es = np.where(g.random(m) < 0.3, g.integers(0, 9, m), g.integers(0, 300_000, m))
    _fused(300_000, m, es, g.permutation(m))


def test_pairs_beyond_the_fused_range(monkeypatch):
    monkeypatch.setattr(P.SmallestPairs, "FUSED_MIN", 0)
    g = np.random.default_rng(4)
    es, is_ = g.integers(0, (1 << 25) + 1, 5000), g.permutation(5000)
    assert not P.SmallestPairs((1 << 25) + 1, 5000, torch.from_numpy(es).to(DEV), torch.from_numpy(is_).to(DEV)).fused
    _run((1 << 25) + 1, 5000, es, is_)


@pytest.mark.parametrize("k", [63, 64, 65, 2047, 2048, 2049, 16384])
def test_fused_pairs_positions_of_a_wave(k, monkeypatch):
    """A wave of the reducing pass takes the runs of 16 chunks as rows of 64
    positions, 2048 marked at a time: k entries of bucket 0 in a chunk, a chunk
    without any, and more chunks than the workgroup's waves take at once."""
    monkeypatch.setattr(P.SmallestPairs, "FUSED_MIN", 0)
    g = np.random.default_rng(k)
    m, verts = 257 * 16384 + 5, 1 << 20
    es = g.integers(verts // 2, verts, m)
    for c in (0, 1, 3, 15, 16, 255, 256):
        es[c * 16384:c * 16384 + k] = g.integers(0, 64, k)
    _fused(verts, m, es, g.permutation(m))


def test_flags_and_positions_of_both_ways(monkeypatch):
    """``flags`` and ``pos`` read the same after a fused run and a step by step one."""
    g = np.random.default_rng(6)
    m, verts = 50_001, 9000
    es = torch.from_numpy(np.where(g.random(m) < 0.1, -3, g.integers(0, verts, m))).to(DEV)
    is_ = torch.from_numpy(g.permutation(2 * m)[:m]).to(DEV)
    step = P.SmallestPairs(verts, m, es, is_)
    monkeypatch.setattr(P.SmallestPairs, "FUSED_MIN", 0)
    fused = P.SmallestPairs(verts, m, es, is_)
    assert fused.fused and not step.fused
    step.run()
    fused.run()
    assert torch.equal(step.flags, fused.flags) and torch.equal(step.pos, fused.pos)
    assert fused.flags.dtype == torch.uint8 and fused.pos.dtype == torch.int64
    assert int(fused.flags.sum()) == int(fused.split) == int(step.split)
