"""The pair bounds computed before the full scan's queue: a search that leaves
out the pairs whose bound exceeds their query's phase-1 bound returns exactly
what the search that scans every pair returns (AMP_PAIR_SKIP=0, which neither
computes nor reads them), at the edges of the bound kernels' tiles: 32 pairs
per tile, 1 to 4 tiles per workgroup, chunks of 16 subspaces, subspace widths
with and without packed row writes, absent probes."""
import numpy as np
import pytest

import paper_2606_07156_amd as amp
from amp_data import random_model

pytestmark = pytest.mark.gpu


def random_index(seed, M, dsub, nlist=40, n=6000, metric="l2", scale=3.0, grid_e=-5):
    """Random arrays in the index format (bounds do not need a trained
    index); list 0 is empty."""
    r = np.random.default_rng(seed)
    d = M * dsub
    cuts = np.sort(r.integers(0, n + 1, nlist - 2))
    off = np.concatenate([[0, 0], cuts, [n]]).astype(np.int64)
    ids = np.concatenate([np.sort(r.choice(10 * n, size=off[p + 1] - off[p], replace=False)) * nlist + p
                          for p in range(nlist)]).astype(np.int64)
    return dict(d=d, M=M, nlist=nlist, metric=metric, grid_kind="u9", grid_e=grid_e,
                centroids=(r.standard_normal((nlist, d)) * scale).astype(np.float32),
                codebook=r.standard_normal((M, 256, dsub)).astype(np.float32), list_offsets=off, ids=ids,
                codes=r.integers(0, 256, (n, M)).astype(np.uint8),
                radq=r.integers(1, 500, nlist).astype(np.int32), list_sizes=np.diff(off).astype(np.int32))


# (pairs, nprobe): one pair, around a tile of 32, ragged tiles, and batches of
# one, two and four tiles per workgroup (from 384 workgroups on)
SIZES = [(1, 1), (31, 31), (33, 11), (257, 1), (24_552, 33), (24_579, 9), (49_152, 12), (66_003, 9)]
# queries with no usable bound (a NaN, squares that overflow) and with squares
# that underflow: the scan decides.  (It finds the pairs of an infinite query
# dead by its own bound, which AMP_PAIR_SKIP=0 turns off: no reference here.)
def odd_queries(Q):
    Q[0, 0], Q[2, 1], Q[3] = np.nan, -1e30, 1e-25
    return Q


SHAPES = [(16, 8), (24, 4), (32, 2), (12, 1), (20, 3), (36, 6), (120, 8)]


@pytest.mark.parametrize("M,dsub", SHAPES)
@pytest.mark.parametrize("policy", ["adaptive", "fixed", "fp32"])
def test_dropping_pairs_by_their_bound_changes_nothing(monkeypatch, M, dsub, policy):
    idx = random_index(M * 10 + dsub, M, dsub)
    h = amp.amp_index_from_arrays(idx)
    amp.amp_index_set_predictor(h, random_model(5, 40, [1500, 0, 0, 0, 0], [60000, 8000, 8000, 8000, 8000]))
    r = np.random.default_rng(M)
    dropped = 0
    for pairs, nprobe in SIZES:
        if M > 100 and pairs > 50_000:
            continue
        nq = pairs // nprobe
        near = r.integers(0, idx["nlist"], nq)
        Q = (idx["centroids"][near] + r.standard_normal((nq, idx["d"]))).astype(np.float32)
        np_q = np.full(nq, nprobe, np.int32)
        np_q[1::3] = np.maximum(1, nprobe // 2)  # absent probes at the end of rows
        kw = dict(policy=policy, want_bits=True, want_probes=True, work=True, **(dict(bits=8) if policy == "fixed" else {}))
        got = amp.amp_search(h, Q, 5, np_q, **kw)
        monkeypatch.setenv("AMP_PAIR_SKIP", "0")
        want = amp.amp_search(h, Q, 5, np_q, **kw)
        monkeypatch.delenv("AMP_PAIR_SKIP")
        for f in ("ids", "dist", "bits", "qdist", "probes"):
            assert np.array_equal(got[f], want[f]), (pairs, f)
        # (a pair of an empty list forms no unit: counted only where dropped)
        empty = np.isin(got["probes"], np.flatnonzero(np.diff(idx["list_offsets"]) == 0)).sum()
        counted = got["work"]["live_pairs"] + got["work"]["dead_pairs"]
        assert np_q.sum() - empty <= counted <= np_q.sum()
        dropped += got["work"]["dead_pairs"]
    assert dropped > 0


@pytest.mark.parametrize("M,dsub", [(16, 8), (20, 3)])
def test_fp32_bounds_of_odd_queries(monkeypatch, M, dsub):
    idx = random_index(3 + M, M, dsub)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M)
    Q = odd_queries((idx["centroids"][r.integers(0, 40, 64)] + r.standard_normal((64, idx["d"]))).astype(np.float32))
    got = amp.amp_search(h, Q, 5, 20, policy="fp32")
    monkeypatch.setenv("AMP_PAIR_SKIP", "0")
    want = amp.amp_search(h, Q, 5, 20, policy="fp32")
    for f in ("ids", "dist"):
        assert np.array_equal(got[f], want[f], equal_nan=f == "dist"), f


@pytest.mark.parametrize("M,dsub", [(8, 4), (16, 5), (96, 8)])
@pytest.mark.parametrize("policy", ["explicit", "fixed"])
def test_dropping_pairs_changes_nothing_under_l1(monkeypatch, M, dsub, policy):
    """The same under L1: 32 pairs per workgroup of the bases."""
    idx = random_index(M + dsub, M, dsub, metric="l1")
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M)
    dropped = 0
    for pairs, nprobe in ((1, 1), (31, 31), (33, 11), (257, 1), (4400, 11)):
        nq = pairs // nprobe
        Q = (idx["centroids"][r.integers(0, idx["nlist"], nq)] + r.standard_normal((nq, idx["d"]))).astype(np.float32)
        np_q = np.full(nq, nprobe, np.int32)
        np_q[1::3] = np.maximum(1, nprobe // 2)
        kw = dict(policy=policy, work=True)
        if policy == "explicit":
            kw["explicit_bits"] = r.choice(np.array([4, 8, 12, 16], np.uint8), size=(nq, nprobe))
        else:
            kw["bits"] = 8
        got = amp.amp_search(h, Q, 5, np_q, **kw)
        monkeypatch.setenv("AMP_PAIR_SKIP", "0")
        want = amp.amp_search(h, Q, 5, np_q, **kw)
        monkeypatch.delenv("AMP_PAIR_SKIP")
        for f in ("ids", "dist", "qdist"):
            assert np.array_equal(got[f], want[f]), (pairs, f)
        dropped += got["work"]["dead_pairs"]
    assert dropped > 0
