"""The nprobe smallest (coarse distance, list) of each query equal a sort of the
returned distances, where the search by bits starts late or cannot end early:
rows of one value, of a few values (ties at the nprobe-th), of both signs, and
rows whose keys share all but their last bits; a wave and a workgroup per query."""
import numpy as np
import pytest

import paper_2606_07156_amd as amp
from test_gpu_pair_bounds import random_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nlist", [2, 63, 64, 65, 250, 700, 1025, 3000])
@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("nq", [3, 2100])
def test_probes_are_a_sort_of_the_distances(nlist, metric, nq):
    idx = random_index(nlist, 8, 2, nlist=nlist, n=2000, metric=metric)
    r = np.random.default_rng(nlist)
    C = idx["centroids"]
    kinds = [C, np.full_like(C, 3.0), C[r.integers(0, min(3, nlist), nlist)],
             (1000 + r.integers(0, 3, C.shape) * 2.0 ** -12).astype(np.float32)]
    Q = (C[r.integers(0, nlist, nq)] + r.standard_normal((nq, idx["d"]))).astype(np.float32)
    Q[0] = 0
    for kind in kinds:
        idx["centroids"] = np.ascontiguousarray(kind, np.float32)
        h = amp.amp_index_from_arrays(idx)
        for nprobe in sorted({1, 2, min(nlist, 31), min(nlist, 64), min(nlist, 100), min(nlist, 256)}):
            if nq > 3 and nprobe > 100:
                continue
            g = amp.amp_search(h, Q, 2, nprobe, policy="fixed", bits=8, want_probes=True, want_coarse=True)
            # (-0 sorts before +0)
            key = g["coarse"].view(np.int32).astype(np.int64)
            key = np.where(key < 0, -1 - (key & 0x7FFFFFFF), key)
            want = np.argsort(key, axis=1, kind="stable")[:, :nprobe]
            assert np.array_equal(g["probes"], want), nprobe
