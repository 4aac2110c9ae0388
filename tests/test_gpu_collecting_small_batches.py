"""Small batches by the collecting scan (asked for; by themselves they go by group maxima): streamed rows, and a few queries whose
candidates do not fit beside ordinary ones.  Needs a real MI355X."""
import pytest
import torch

from paper_2110_08919_amd import lpq, synth

pytestmark = pytest.mark.gpu


def _same(got, want):
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.fixture
def collecting():
    lpq.set_tuning(lpq.TUNE_PATH, 3)
    yield
    lpq.set_tuning(lpq.TUNE_PATH, 0)


@pytest.mark.parametrize("n,d,nq,k,metric", [
    (12_000, 600, 64, 10, "l2sq"), (12_000, 600, 1, 10, "ip"), (30_000, 1024, 100, 10, "ip"), (20_000, 2048, 128, 20, "l2sq"),
    (9000, 4096, 257, 3, "ip"), (40_009, 300, 33, 100, "l2sq"), (100_000, 100, 64, 100, "l2sq"), (70_000, 200, 16, 10, "ip"),
])
def test_same_results(collecting, n, d, nq, k, metric):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    x, q = (torch.randn((m, d), generator=g, device="cuda") for m in (n, nq))
    index = lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "absmax", "global"), n).add_f32(x)
    assert lpq.search_plan_info(d, 8, False, n, nq, k)[0] == 3 and not any(lpq.search_maxima_info(d, 8, False, n, nq, k))
    got = index.search(q, k, metric)
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    want = index.search(q, k, metric)
    lpq.set_tuning(lpq.TUNE_PATH, 3)
    torch.cuda.synchronize()
    _same(got, want)


@pytest.mark.parametrize("n,d,nq,k,flagged", [(60_000, 100, 20, 100, 2), (60_000, 100, 64, 20, 30), (60_000, 200, 40, 100, 5)])
def test_a_few_queries_are_searched_again(collecting, n, d, nq, k, flagged):
    w = synth.Workload("w", "bimodal", n, d, nq, "l2sq", (k,), "minmax", "global", 3)
    x, q = w.corpus("cuda"), w.queries("cuda")
    gq = lpq.Quantizer(d, 8).calibrate(x, "minmax", "global")
    x[torch.randperm(n, generator=torch.Generator().manual_seed(1))[: n // 3].cuda()] = x[0].clone()
    index = lpq.Index(gq, n).add_f32(x)
    some = torch.unique((torch.arange(flagged) * 617 + 3) % nq).cuda()
    q[some] = x[0]
    assert not any(lpq.search_maxima_info(d, 8, False, n, nq, k))
    got = index.search(q, k, "l2sq")
    torch.cuda.synchronize()
    redone, fill = index.overflow_stats(nq, k, "l2sq")
    assert redone >= len(some) and fill > 0
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    want = index.search(q, k, "l2sq")
    lpq.set_tuning(lpq.TUNE_PATH, 3)
    torch.cuda.synchronize()
    _same(got, want)
