"""A handful of queries whose candidates do not fit beside a batch of ordinary ones: an item stored many
times over ties with itself at their bound.  Up to 8 or 16 of them in a large batch go to the generic
kernel, more of them through further rounds of the scan.  Needs a real MI355X."""
import pytest
import torch

from paper_2110_08919_amd import lpq, synth

pytestmark = pytest.mark.gpu


# both sides of the limits (8 from 2048 queries on, 16 from 8192 on, none below or beyond 32 results), scans of
# long and of streamed rows and of short ones with lists the register kernel does not take
@pytest.mark.parametrize("n,d,nq,k,flagged", [
    (30_000, 300, 2047, 10, 3), (30_000, 300, 2048, 10, 1), (30_000, 300, 2048, 10, 8), (30_000, 300, 2100, 10, 9),
    (20_000, 800, 8192, 5, 16), (20_000, 800, 8200, 5, 17), (40_000, 64, 9000, 32, 16), (40_000, 64, 3000, 33, 4),
    (40_000, 64, 2500, 20, 40), (60_000, 100, 700, 100, 5), (60_000, 100, 20, 100, 2),
])
def test_a_few_queries_are_searched_again(n, d, nq, k, flagged):
    w = synth.Workload("w", "bimodal", n, d, nq, "l2sq", (k,), "minmax", "global", 3)
    x, q = w.corpus("cuda"), w.queries("cuda")
    gq = lpq.Quantizer(d, 8).calibrate(x, "minmax", "global")
    rows = torch.randperm(n, generator=torch.Generator().manual_seed(1))[: n // 3].cuda()
    x[rows] = x[0].clone()
    index = lpq.Index(gq, n).add_f32(x)
    some = torch.unique((torch.arange(flagged) * 617 + 3) % nq).cuda()
    q[some] = x[0]
    for metric in ("l2sq", "ip"):
        got = index.search(q, k, metric)
        torch.cuda.synchronize()
        if metric == "l2sq":
            assert index.overflow_stats(nq, k, metric)[0] >= len(some)
        lpq.set_tuning(lpq.TUNE_PATH, 1)
        try:
            want = index.search(q, k, metric)
            torch.cuda.synchronize()
        finally:
            lpq.set_tuning(lpq.TUNE_PATH, 0)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("n,d,nq,k,bits", [(6216, 20, 200, 21, 3), (8000, 60, 64, 30, 3), (8300, 60, 65, 12, 4)])
def test_packed_tiles_with_thousands_of_ties(n, d, nq, k, bits):
    """Tiles of 64 queries with up to and beyond 256 regions, most items equal at the bound."""
    w = synth.Workload("w", "skewed_int", n, d, nq, "ip", (k,), "absmax", "per_feature", 1)
    x, q = w.corpus("cuda"), w.queries("cuda")
    index = lpq.Index(lpq.Quantizer(d, bits).calibrate(x, "absmax", "per_feature"), n, packed=True).add_f32(x)
    got = index.search(q, k, "ip")
    torch.cuda.synchronize()
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want = index.search(q, k, "ip")
        torch.cuda.synchronize()
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
