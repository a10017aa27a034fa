"""Small batches take fused launches (one workgroup builds the work queue, one
kernel each bounds and merges); a query's results must not depend on it.  Rows
of one large batch (general launches) against the same queries in batches on
either side of each limit: 4096 pairs, 512 queries, 5120 lists; k above the
list sizes, so that the bound spans several probes; lists split in chunks;
device-resident sizes up to and beyond the 8192 queries one workgroup clamps."""
import numpy as np
import pytest

import paper_2606_07156_amd as amp
from test_gpu_pair_bounds import random_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policy,bits", [("fixed", 8), ("explicit", 0), ("fp32", 0)])
@pytest.mark.parametrize("nlist,metric", [(40, "l2"), (5120, "l2"), (5121, "ip"), (300, "ip")])
def test_rows_of_small_and_large_batches_agree(monkeypatch, policy, bits, nlist, metric):
    idx = random_index(nlist, 8, 4, nlist=nlist, n=20_000, metric=metric)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(nlist)
    nq, nprobe, k = 1030, 8, 70
    Q = (idx["centroids"][r.integers(0, nlist, nq)] + r.standard_normal((nq, 32))).astype(np.float32)
    xb = r.choice(np.array([4, 8, 12, 16], np.uint8), size=(nq, nprobe))
    kw = dict(policy=policy, bits=bits or 16)

    def search(a, b):
        x = dict(explicit_bits=xb[a:b]) if policy == "explicit" else {}
        return amp.amp_search(h, Q[a:b], k, nprobe, **kw, **x)

    want = search(0, nq)
    for a, n in ((0, 1), (3, 33), (100, 512), (17, 513)):  # 8, 264, 4096 and 4104 pairs
        for chunk in ("", "256"):
            monkeypatch.setenv("AMP_CHUNK", chunk)
            monkeypatch.setenv("AMP_CHUNK1", chunk)
            got = search(a, a + n)
            for f in ("ids", "dist", "qdist"):
                assert np.array_equal(got[f], want[f][a:a + n]), (a, n, chunk, f)
        monkeypatch.delenv("AMP_CHUNK")
        monkeypatch.delenv("AMP_CHUNK1")


@pytest.mark.parametrize("nq", [5, 8192, 8193])
def test_device_sizes_are_clamped_by_one_or_many_workgroups(nq):
    import torch
    idx = random_index(3, 8, 4)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(nq)
    Q = (idx["centroids"][r.integers(0, 40, nq)] + r.standard_normal((nq, 32))).astype(np.float32)
    k, p = r.integers(1, 6, nq).astype(np.int32), r.integers(1, 4, nq).astype(np.int32)
    dev = "cuda:0"
    out = dict(ids=torch.empty((nq, 5), dtype=torch.int64, device=dev),
               dist=torch.empty((nq, 5), dtype=torch.float32, device=dev),
               status=torch.full((1,), 7, dtype=torch.int32, device=dev))
    k[-1] = 5  # the largest size, so that the host search's rows have the same width
    want = amp.amp_search(h, Q, k, p, policy="fixed", bits=8)
    kd, pd = torch.from_numpy(k).to(dev), torch.from_numpy(p).to(dev)
    for last, status in ((9, amp.AMP_EINVAL), (5, amp.AMP_OK)):
        kd[-1] = last  # above kmax: clamped and reported
        torch.cuda.synchronize()
        amp.amp_search(h, torch.from_numpy(Q).to(dev), kd, pd, kmax=5, npmax=int(p.max()), out=out, policy="fixed",
                       bits=8)
        torch.cuda.synchronize()
        assert int(out["status"]) == status
        assert np.array_equal(out["ids"].cpu().numpy(), want["ids"])
        assert np.array_equal(out["dist"].cpu().numpy(), want["dist"])


# buckets of the general queue (FP32 policy: one per list) around those that its
# scan holds in registers, one to four per thread, and beyond
@pytest.mark.parametrize("nlist", [100, 1023, 1024, 1025, 3073, 4096, 4097])
def test_general_queue_at_edges_of_its_scan(nlist):
    idx = random_index(nlist, 8, 4, nlist=nlist, n=20_000)
    h = amp.amp_index_from_arrays(idx)
    r = np.random.default_rng(nlist)
    Q = (idx["centroids"][r.integers(0, nlist, 600)] + r.standard_normal((600, 32))).astype(np.float32)
    want = amp.amp_search(h, Q, 10, 8, policy="fp32")  # 4800 pairs
    for a in (0, 299, 500):
        got = amp.amp_search(h, Q[a:a + 100], 10, 8, policy="fp32")  # the small queue
        for f in ("ids", "dist"):
            assert np.array_equal(got[f], want[f][a:a + 100]), (a, f)
