"""The scan's lane classes around the subspace counts where they change: 16-bit
lanes up to M = 16, byte entries for the 8-bit pairs of 17 to 128 subspaces,
16-bit entries with 32-bit sums for every wider pair; bit-exact against the
oracle, single widths and mixed ones, few and many pairs per list, and with
codes that reach the largest sums (every entry of a row at the width's top)."""
import numpy as np
import pytest

import oracle
import paper_2606_07156_amd as amp
from _parity import compare_integer
from test_gpu_pair_bounds import random_index

pytestmark = pytest.mark.gpu


def _largest_sums(idx, M):
    # codeword 255 lies far from every residual: a vector of 255s takes the top
    # entry of every row
    idx["codebook"][:, 255] = 40.0
    idx["grid_e"] = -2
    idx["codes"][::7] = 255
    return idx


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("M", [16, 20, 24, 96, 128, 132])
@pytest.mark.parametrize("bits", [4, 8, 12, 16, 0])
def test_lane_classes_are_bit_exact(metric, M, bits):
    idx = _largest_sums(random_index(M + 7, M, 2, nlist=12, n=1500, metric=metric), M)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M + bits)
    for nq, nprobe, k in ((9, 12, 300), (40, 5, 3)):
        Q = (idx["centroids"][r.integers(0, 12, nq)] + r.standard_normal((nq, 2 * M))).astype(np.float32)
        kw = dict(policy="fixed", bits=bits)
        if bits == 0:
            kw = dict(policy="explicit", explicit_bits=r.choice(np.array([4, 8, 12, 16], np.uint8), size=(nq, nprobe)))
        g = amp.amp_search(h, Q, k, nprobe, want_probes=True, **kw)
        compare_integer(g, oracle.search(idx, Q, k, nprobe, probes=g["probes"], **kw))


# L1's row ranges: sixteen lanes per (pair, subspace) row, fewer rows than a
# workgroup has groups of sixteen, and more
@pytest.mark.parametrize("M,dsub", [(4, 8), (8, 4), (16, 5), (24, 2), (36, 3), (96, 2), (132, 1)])
@pytest.mark.parametrize("bits", [4, 8, 12, 16, 0])
def test_lane_classes_under_l1_are_bit_exact(M, dsub, bits):
    idx = random_index(M + 9, M, dsub, nlist=12, n=1500, metric="l1")
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M + bits)
    for nq, nprobe, k in ((1, 1, 5), (40, 5, 3)):
        Q = (idx["centroids"][r.integers(1, 12, nq)] + r.standard_normal((nq, idx["d"]))).astype(np.float32)
        kw = dict(policy="fixed", bits=bits)
        if bits == 0:
            kw = dict(policy="explicit", explicit_bits=r.choice(np.array([4, 8, 12, 16], np.uint8), size=(nq, nprobe)))
        g = amp.amp_search(h, Q, k, nprobe, want_probes=True, **kw)
        compare_integer(g, oracle.search(idx, Q, k, nprobe, probes=g["probes"], **kw))
