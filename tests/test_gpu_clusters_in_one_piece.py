"""Corpora stored cluster by cluster: the rows near a query lie in few stages of the scan, in few groups of its sample and in few
regions.  The further rounds leave nothing to the generic kernel, and the results are its.  Needs a real MI355X."""
import pytest
import torch

from paper_2110_08919_amd import lpq

pytestmark = pytest.mark.gpu


def _clusters(n, d, nq, run, noise, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    c = torch.randn((n // run + 1, d), generator=g, device="cuda")
    x = c.repeat_interleave(run, 0)[:n] + noise * torch.randn((n, d), generator=g, device="cuda")
    q = c[torch.randint(0, n // run, (nq,), generator=g, device="cuda")] + noise * torch.randn((nq, d), generator=g, device="cuda")
    return x, q


@pytest.mark.parametrize("n,d,nq,k,run,metric", [
    (79_076, 541, 4465, 100, 439, "l2sq"), (168_405, 74, 8080, 200, 468, "l2sq"), (56_000, 300, 2000, 40, 200, "ip"), (100_000, 128, 1000, 10, 700, "l2sq"),
])
def test_large_batches(n, d, nq, k, run, metric):
    x, q = _clusters(n, d, nq, run, 0.3, n)
    index = lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "minmax", "global"), n).add_f32(x)
    ws = torch.empty(index.workspace_bytes(nq, k, metric) + 256, dtype=torch.uint8, device="cuda")
    ids, dists = index.search(q, k, metric, workspace=ws)
    torch.cuda.synchronize()
    assert index.overflow_left(nq, k, metric, ws) <= nq // 100
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q[::16].contiguous(), k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists[::16], want) and torch.equal(ids[::16], want_ids)


# group maxima by workgroups of 1024 threads (streamed rows, and many groups) and of 256
@pytest.mark.parametrize("n,d,nq,k,run,metric", [
    (57_474, 667, 427, 10, 1646, "l2sq"), (95_962, 856, 5, 100, 2463, "ip"), (5600, 512, 3, 21, 700, "l2sq"), (700_001, 64, 4, 30, 3000, "ip"),
    (1_100_000, 128, 2, 128, 5000, "l2sq"), (50_048, 100, 200, 10, 400, "l2sq"),
])
def test_small_batches(n, d, nq, k, run, metric):
    assert lpq.search_maxima_info(d, 8, False, n, nq, k)[0] > 0
    x, q = _clusters(n, d, nq, run, 0.25, n)
    index = lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "minmax", "global"), n).add_f32(x)
    ids, dists = index.search(q, k, metric)
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q, k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists, want) and torch.equal(ids, want_ids)
