"""The width predictor's sum over support vectors, against the oracle: numbers
of support vectors at the edges of a step (four records per thread when a
thread has a whole pair, eight per thread when several share one, none at all),
and gammas on both sides of the 24-bit table-index product (g_mul 2^24)."""
import numpy as np
import pytest

import oracle
import paper_2606_07156_amd as amp
from amp_data import random_model
from test_gpu_pair_bounds import random_index
from test_gpu_parity import _dq2

pytestmark = pytest.mark.gpu

NPROBE = 4


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("gamma", [0.03, 1.0, 40.0, 900.0])
def test_widths_are_the_oracles(metric, gamma):
    idx = random_index(7, 16, 4, metric=metric)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(3)
    # 33k queries of four probes: a thread per pair; 6 queries: 64 threads per pair
    Q = (idx["centroids"][r.integers(0, idx["nlist"], 33_000)]
         + r.standard_normal((33_000, idx["d"]))).astype(np.float32)
    few = amp.amp_search(h, Q[:6], 4, NPROBE, policy="fixed", bits=8, want_probes=True)["probes"]
    dq = [_dq2(idx, q, P) for q, P in zip(Q, few)]
    feats = [np.concatenate(dq), idx["radq"], idx["radq"], idx["list_sizes"], idx["list_sizes"]]
    logs = [oracle.mitchell_log2_q8(np.asarray(f, np.int64)) for f in feats]
    lo = [int(L.min()) for L in logs]
    mul = [int(1023 * 65536 // max(1, int(L.max() - L.min()))) for L in logs]
    for n_sv in [0, 1, 3, 4, 5, 7, 8, 63, 65, 511, 513]:
        m = random_model(n_sv, n_sv, lo, mul, gamma=gamma)
        ys = [oracle.predict_pair_bits(D, P, idx["radq"], idx["list_sizes"], m)[1] for D, P in zip(dq, few)]
        # thresholds at scores that occur: a sum off by one changes a width
        m["theta"] = np.sort(np.concatenate(ys).astype(np.int64))[[5, 11, 17]]
        amp.amp_index_set_predictor(h, m)
        want = np.stack([oracle.predict_pair_bits(D, P, idx["radq"], idx["list_sizes"], m)[0]
                         for D, P in zip(dq, few)])
        a = amp.amp_search(h, Q[:6], 4, NPROBE, policy="adaptive", want_bits=True, want_probes=True)
        b = amp.amp_search(h, Q, 4, NPROBE, policy="adaptive", want_bits=True, want_probes=True)
        assert np.array_equal(a["probes"], few) and np.array_equal(b["probes"][:6], few)
        assert np.array_equal(a["bits"], want.astype(np.uint8))
        assert np.array_equal(b["bits"][:6], want.astype(np.uint8))
