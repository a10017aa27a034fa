"""Inner product's tables per query.  Integer policies: the table build split
over subspaces gives the answers of the oracle (a few queries) and of the unsplit
build (a batch that fills the chip), at numbers of subspaces that a split does
not divide.  FP32 policy: the pairs left out by the bound from the coarse
distance change nothing, at every subspace width, at edges of the table
kernel's groups of four and 32 queries, for data far from the origin (where the
bound's slack is large against the distances' differences) and odd queries; the scan that copies
its LUT from the table agrees with FP64, at every number of its steps of 64
subspaces; so does the bound that integer cluster locating leaves to the rows
themselves."""
import numpy as np
import pytest

import oracle
import paper_2606_07156_amd as amp
from _parity import compare_fp32
from test_gpu_pair_bounds import random_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,dsub", [(4, 8), (8, 8), (20, 3), (36, 4), (96, 8), (120, 8)])
@pytest.mark.parametrize("gran", ["pair", "subspace"])
def test_split_table_build(M, dsub, gran):
    idx = random_index(M, M, dsub, metric="ip", n=3000)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M)
    Q = (idx["centroids"][r.integers(1, 40, 4100)] + r.standard_normal((4100, idx["d"]))).astype(np.float32)
    kw = dict(policy="fixed", bits=8, granularity=gran, want_probes=True)
    full = amp.amp_search(h, Q, 10, 6, **kw)  # 513 groups of eight: one workgroup each
    for nq in (1, 9):
        part = amp.amp_search(h, Q[:nq], 10, 6, **kw)
        for f in ("ids", "dist", "qdist", "probes"):
            assert np.array_equal(part[f], full[f][:nq]), (nq, f)
    if gran == "pair":
        ref = oracle.search(idx, Q[:3], 10, 6, policy="fixed", bits=8, probes=full["probes"][:3])
        assert np.array_equal(full["ids"][:3], ref["ids"])


@pytest.mark.parametrize("M,dsub", [(16, 8), (24, 7), (8, 6), (32, 5), (24, 4), (20, 3), (36, 2), (12, 1), (96, 8)])
@pytest.mark.parametrize("offset", [0.0, 30.0])
def test_fp32_bound_from_the_coarse_distance(monkeypatch, M, dsub, offset):
    idx = random_index(M + dsub, M, dsub, metric="ip")
    idx["centroids"] = (idx["centroids"] + offset).astype(np.float32)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M)
    dead = 0
    for nq in (1, 5, 31, 33, 700):
        Q = (idx["centroids"][r.integers(0, 40, nq)] + r.standard_normal((nq, idx["d"]))).astype(np.float32)
        if nq == 33:
            Q[2, 1], Q[3] = -1e30, 1e-25  # no usable bound, squares that underflow
        np_q = np.full(nq, 12, np.int32)
        np_q[1::3] = 5
        got = amp.amp_search(h, Q, 5, np_q, policy="fp32", work=True)
        monkeypatch.setenv("AMP_PAIR_SKIP", "0")
        want = amp.amp_search(h, Q, 5, np_q, policy="fp32")
        monkeypatch.delenv("AMP_PAIR_SKIP")
        for f in ("ids", "dist"):
            assert np.array_equal(got[f], want[f], equal_nan=f == "dist"), (nq, f)
        dead += got["work"]["dead_pairs"]
    assert dead > 0


@pytest.mark.parametrize("M", [12, 64, 68, 100, 128, 132, 152])
def test_fp32_scan_of_copied_tables(M):
    idx = random_index(M, M, 2, metric="ip", n=3000)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M)
    Q = (idx["centroids"][r.integers(1, 40, 20)] + r.standard_normal((20, idx["d"]))).astype(np.float32)
    got = amp.amp_search(h, Q, 10, 12, policy="fp32", want_probes=True)
    compare_fp32(got, oracle.search(idx, Q, 10, 12, policy="fp32", probes=got["probes"]), idx, Q)


@pytest.mark.parametrize("M,dsub", [(16, 8), (36, 4), (96, 8)])
def test_fp32_bound_under_integer_cluster_locating(monkeypatch, M, dsub):
    idx = random_index(M + 1, M, dsub, metric="ip")
    h = amp.amp_index_from_arrays(idx)
    amp.amp_index_build_cl_map(h, M // 4, 8, iters=4, seed=2)
    r = np.random.default_rng(M)
    Q = (idx["centroids"][r.integers(0, 40, 70)] + r.standard_normal((70, idx["d"]))).astype(np.float32)
    kw = dict(policy="fp32", cl_policy="fixed", cl_bits=8, want_probes=True)
    got = amp.amp_search(h, Q, 5, 20, work=True, **kw)
    monkeypatch.setenv("AMP_PAIR_SKIP", "0")
    want = amp.amp_search(h, Q, 5, 20, **kw)
    for f in ("ids", "dist", "probes"):
        assert np.array_equal(got[f], want[f]), f
    assert got["work"]["dead_pairs"] > 0
    compare_fp32(got, oracle.search(idx, Q, 5, 20, policy="fp32", probes=got["probes"]), idx, Q)


def test_fp32_tables_beyond_the_y_limit_of_a_grid(monkeypatch):
    """65535 groups of 32 queries, which is as many workgroups as y may have, and
    one group more."""
    monkeypatch.setenv("AMP_CAPQ", "64")
    idx = random_index(3, 12, 1, nlist=8, n=200, metric="ip")
    h = amp.amp_index_from_arrays(idx)
    last = 65535 * 32
    Q = np.random.default_rng(3).standard_normal((last + 5, 12)).astype(np.float32)
    got = amp.amp_search(h, Q, 5, 2, policy="fp32")
    for at in (slice(0, 40), slice(last - 35, last + 5)):
        want = amp.amp_search(h, Q[at], 5, 2, policy="fp32")
        for f in ("ids", "dist"):
            assert np.array_equal(got[f][at], want[f]), (at, f)
