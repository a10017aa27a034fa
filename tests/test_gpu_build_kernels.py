"""One k-means update of the index build, exactly: on small-integer data every
FP32 distance is exact, so the nearest centroid (ties to the lower index) and
the mean FP64 sum * (1 / count) are known bit for bit.  Subspace widths 1 to 8,
row counts around the kernels' 16-, 64- and 1024-row tiles, one and two sort
passes (more than 256 clusters), and codebooks with fewer distinct rows than
codewords (clusters that run empty)."""
import numpy as np
import pytest

import paper_2606_07156_amd as amp

pytestmark = pytest.mark.gpu


def _update(X, C0):
    D = ((X[:, None, :] - C0[None]) ** 2).sum(2)
    a = D.argmin(1)
    out, n = C0.copy(), np.bincount(a, minlength=len(C0))
    for c in np.flatnonzero(n):
        out[c] = X[a == c].sum(0) * (1.0 / n[c])
    return out.astype(np.float32), n > 0


def _seeded_order(n, seed):
    """The build's order of training rows: by SplitMix64 of the row number."""
    with np.errstate(over="ignore"):
        x = (np.uint64(seed) + np.uint64(0x5851F42D4C957F2D)) ^ np.arange(n, dtype=np.uint64)
        x += np.uint64(0x9E3779B97F4A7C15)
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return np.argsort(x ^ (x >> np.uint64(31)), kind="stable")


@pytest.mark.parametrize("dsub", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("n", [520, 1025, 2063])
def test_codebook_update(dsub, n):
    # integer data: the centroids are rounded, so the residuals are integers
    M, nlist, seed = 4, 9, n + dsub
    r = np.random.default_rng(seed)
    base = r.integers(-60, 61, size=(n, M * dsub)).astype(np.float32)
    ix = amp.amp_index_get_arrays(amp.amp_index_build(base, nlist, M, iters=1, seed=seed, integer_data=True))
    rows, lst = ix["ids"], np.repeat(np.arange(nlist), np.diff(ix["list_offsets"]))
    R = np.empty_like(base)
    R[rows] = base[rows] - ix["centroids"][lst]
    for m in range(M):
        X = R[:, m * dsub:(m + 1) * dsub].astype(np.float64)
        first = list(dict.fromkeys(map(tuple, X[_seeded_order(n, seed + 1000 + m)])))[:256]
        first = np.array([first[i % len(first)] for i in range(256)])
        want, full = _update(X, first)
        assert np.array_equal(ix["codebook"][m][full], np.rint(want[full])), m
        assert full.all() or dsub <= 2


@pytest.mark.parametrize("n,nlist", [(700, 16), (5003, 300), (3000, 2049)])
def test_coarse_update(n, nlist):
    r = np.random.default_rng(n)
    base = r.integers(-30, 31, size=(n, 16)).astype(np.float32)
    C0 = amp.amp_index_get_arrays(amp.amp_index_build(base, nlist, 4, iters=0, seed=n))["centroids"]
    C1 = amp.amp_index_get_arrays(amp.amp_index_build(base, nlist, 4, iters=1, seed=n))["centroids"]
    want, full = _update(base.astype(np.float64), C0.astype(np.float64))
    assert full.all() and np.array_equal(C1, want)
