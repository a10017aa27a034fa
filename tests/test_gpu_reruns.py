"""Re-runs of the full scan after a candidate overflow: work units of one pair
and one list chunk, the lane class taken from the pair's width, pairs beyond the
tightened bound left out.  A search whose queries overflow a 256-entry candidate
buffer, once and again, returns exactly what the same search returns with room
for every candidate: every lane class alone and mixed in a query, FP32 tables
computed and copied, lists of one chunk and of several."""
import numpy as np
import pytest

import paper_2606_07156_amd as amp
from test_gpu_pair_bounds import random_index

pytestmark = pytest.mark.gpu

NEAR, LISTS = 40, 60


def _index(metric, M):
    """Forty lists of 150 vectors with like distances, then twenty ever farther
    ones, some of which only a tightened bound leaves out.  A query of k = 48 has
    about 40 x 48 candidates below its phase-1 bound.  The k-th of any 256 of them
    leaves 48 / 256: some 360, give or take 50, beyond the buffer again for most of
    48 queries; that of the next 256 leaves some 70, give or take 15.  So both
    rounds take place and two are enough whatever candidates come first.  4-bit
    tables are coarse: their estimates lie lower, and which pairs come first
    decides how many remain.  With them k = 24, and one round may be enough."""
    idx = random_index(M, M, 2, nlist=LISTS, n=150 * LISTS, metric=metric, scale=0.05)
    idx["list_offsets"] = (np.arange(LISTS + 1) * 150).astype(np.int64)
    idx["list_sizes"] = np.diff(idx["list_offsets"]).astype(np.int32)
    idx["ids"] = np.random.default_rng(M).permutation(150 * LISTS).astype(np.int64).reshape(LISTS, 150)
    idx["ids"] = np.sort(idx["ids"], axis=1).reshape(-1)
    step = np.linspace(0.0, 4.0, LISTS - NEAR)[:, None]
    idx["centroids"][NEAR:] -= step.astype(np.float32)  # (away from the queries' mean)
    return idx


@pytest.mark.parametrize("metric", ["l2", "ip"])
@pytest.mark.parametrize("M", [16, 24, 96])
@pytest.mark.parametrize("policy", ["fixed4", "fixed8", "fixed16", "explicit", "fp32"])
def test_overflows_are_resolved_exactly(monkeypatch, capfd, metric, M, policy):
    idx = _index(metric, M)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(M + 1)
    Q = (0.5 + r.standard_normal((48, 2 * M))).astype(np.float32)
    kw = dict(policy=policy)
    if policy.startswith("fixed"):
        kw = dict(policy="fixed", bits=int(policy[5:]))
    elif policy == "explicit":
        kw["explicit_bits"] = r.choice(np.array([4, 8, 12, 16], np.uint8), size=(48, LISTS))
    coarse = policy in ("fixed4", "explicit")
    k, rounds = (24, "1") if coarse else (48, "1 1")
    want = amp.amp_search(h, Q, k, LISTS, **kw)
    monkeypatch.setenv("AMP_STATS", "1")
    monkeypatch.setenv("AMP_CAPQ", "256")
    for chunk in ("", "64"):  # whole lists; three chunks each
        monkeypatch.setenv("AMP_CHUNK", chunk)
        capfd.readouterr()
        got = amp.amp_search(h, Q, k, LISTS, **kw)
        err = capfd.readouterr().err
        assert f"phase-2 re-runs: {rounds}" in err, err
        for f in ("ids", "qdist", "dist"):
            assert np.array_equal(got[f], want[f]), (chunk, f)
