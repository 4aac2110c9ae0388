"""Small batches by group maxima (three launches): both metrics, row lengths of all kinds of workgroup, packed rows, rows left
over behind the last whole stage, one and many groups to a split, every limit of k and batch, and more groups at the bound
than a workgroup works off at a time (few distinct vectors).  Against the generic kernel.  Needs a real MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(x, q, k, metric, bits=8, packed=False):
    from paper_2110_08919_amd import lpq
    n, d = x.shape
    quant = lpq.Quantizer(d, bits).calibrate(x, "absmax", "global")
    index = lpq.Index(quant, n, packed=packed).add_f32(x)
    ids, dists = index.search(q, k, metric)
    again = index.search(q, k, metric)
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q, k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists, want) and torch.equal(ids, want_ids)
    assert torch.equal(again[0], ids) and torch.equal(again[1], dists)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [
    (4096, 24, 1, 1), (4223, 64, 3, 10), (10_000, 128, 64, 128), (65_535, 96, 16, 10), (70_001, 100, 63, 33), (200_129, 128, 5, 100),
    (300_000, 40, 64, 2), (131_072, 192, 7, 10), (131_135, 256, 64, 100), (9000, 200, 1, 128), (1_000_000, 128, 1, 10),
    (2_000_003, 33, 2, 17),
    # streamed rows: one, two and four loads to a lane of the last kernel
    (4096, 384, 5, 16), (70_001, 300, 64, 100), (66_000, 512, 1, 10), (100_255, 700, 16, 10), (50_007, 1024, 33, 128), (30_300, 1500, 64, 20),
    (40_001, 2048, 9, 10), (20_100, 2100, 64, 33), (12_345, 4000, 3, 40),
])
def test_small_batches(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(n)
    _check(*(torch.randn((m, d), generator=g, device="cuda") for m in (n, nq)), k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(50_000, 64, 40, 10), (100_001, 96, 64, 64), (70_000, 200, 2, 128)])
def test_packed_rows(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(n)
    _check(*(torch.randn((m, d), generator=g, device="cuda") for m in (n, nq)), k, metric, bits=4, packed=True)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,distinct,nq,k", [(100_000, 1, 1, 100), (100_000, 7, 20, 10), (150_000, 900, 64, 30), (60_000, 0, 3, 10)])
def test_many_groups_at_the_bound(metric, n, distinct, nq, k):
    g = torch.Generator(device="cuda").manual_seed(n + distinct)
    if distinct:
        x = torch.randn((distinct, 32), generator=g, device="cuda")[torch.randint(0, distinct, (n,), generator=g, device="cuda")].contiguous()
    else:            # two values to a feature
        x = torch.randint(0, 2, (n, 32), generator=g, device="cuda").float()
    _check(x, x[: nq].clone(), k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
def test_many_groups_of_streamed_rows_at_the_bound(metric):
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((11, 600), generator=g, device="cuda")[torch.randint(0, 11, (40_000,), generator=g, device="cuda")].contiguous()
    _check(x, x[:20].clone(), 10, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(300_001, 64, 16, 10), (400_000, 32, 1, 100), (100_000, 300, 5, 10), (60_000, 16, 64, 20), (10_000, 128, 100, 10), (5003, 64, 3, 128)])
def test_corpora_of_repeated_and_sparse_rows(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn((n, d), generator=g, device="cuda")
    q = x[1:2 * nq:2].clone()
    x[::2] = 0.0                                          # every second row the same
    q[: nq // 2] = 0.0
    _check(x, q, k, metric)
    x = (torch.rand((n, d), generator=g, device="cuda") < 0.05).float()
    _check(x, (torch.rand((nq, d), generator=g, device="cuda") < 0.05).float(), k, metric)
