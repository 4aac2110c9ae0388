"""Searches that go by group maxima, and say so: the largest k on few rows, odd sizes, one and many tiles of queries of every row
length, rows and keys that tie, tied rows that come late, behind the last whole stage only or beside many better ones.  Against
the generic kernel.  Needs a real MI355X."""
import pytest
import torch

from paper_2110_08919_amd import lpq

pytestmark = pytest.mark.gpu


def _same_as_generic(index, q, k, metric):
    ids, dists = index.search(q, k, metric)
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q, k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists, want) and torch.equal(ids, want_ids)


def _check(x, q, k, metric):
    n, d = x.shape
    assert lpq.search_maxima_info(d, 8, False, n, q.shape[0], k)[0] > 0, "group maxima were expected here"
    _same_as_generic(lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "absmax", "global"), n).add_f32(x), q, k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(33_100, 128, 64, 128), (65_407, 96, 16, 10), (40_009, 200, 1, 128)])
def test_few_rows(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    _check(*(torch.randn((m, d), generator=g, device="cuda") for m in (n, nq)), k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [
    # two, three and many tiles of 64 queries: the limits of each, rows of two and four waves, workgroups of 256 and 1024
    (20_577, 100, 65, 10), (10_300, 64, 128, 40), (60_000, 128, 129, 1), (20_500, 24, 192, 10), (5200, 128, 513, 3), (4096, 60, 2048, 5),
    (20_577, 192, 65, 10), (40_100, 256, 128, 33), (20_600, 200, 200, 10),
    # streamed rows
    (30_000, 300, 65, 10), (20_100, 512, 129, 20), (9000, 700, 512, 1), (30_001, 1024, 257, 10), (16_500, 2000, 100, 10),
])
def test_batches_of_several_tiles(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(n)
    _check(*(torch.randn((m, d), generator=g, device="cuda") for m in (n, nq)), k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(33_100, 64, 3, 128), (20_223, 64, 300, 10), (70_001, 200, 16, 10)])
def test_repeated_and_sparse_rows(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn((n, d), generator=g, device="cuda")
    x[::2] = 0.0
    q = torch.randn((nq, d), generator=g, device="cuda")
    q[0] = 0.0
    _check(x, q, k, metric)
    x = (torch.rand((n, d), generator=g, device="cuda") < 0.05).float()
    _check(x, (torch.rand((nq, d), generator=g, device="cuda") < 0.05).float(), k, metric)


def _codes(n, d, nq, seed, high):
    """Whole numbers that are the codes, so that keys tie and differ by one as they are meant to."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randint(0, high, (m, d), generator=g, device="cuda").float() for m in (n, nq))


def _check_codes(x, q, k, metric):
    n, d = x.shape
    quant = lpq.Quantizer(d, 8)
    quant.set_params([0.0] * d, [-128.0] * d, [128.0] * d)
    assert lpq.search_maxima_info(d, 8, False, n, q.shape[0], k)[0] > 0, "group maxima were expected here"
    _same_as_generic(lpq.Index(quant, n).add_f32(x), q, k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(100_001, 64, 16, 10), (70_100, 100, 1, 128), (300_077, 200, 16, 33), (20_223, 64, 300, 10), (60_255, 300, 20, 10),
                                      (40_100, 2048, 130, 5)])
def test_keys_that_tie_and_keys_one_apart(metric, n, d, nq, k):
    """Rows of odd and of even norm at the same E, few of the better ones among many of the others."""
    x, q = _codes(n, d, nq, n, 2)
    x *= (torch.arange(d, device="cuda") < 12).float()
    q *= (torch.arange(d, device="cuda") < 12).float()
    q[0] = 0.0
    _check_codes(x, q, k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k,start", [
    (1_000_000, 32, 16, 10, 0.6), (1_000_000, 32, 1, 100, 0.99),          # the tied rows come late: looks as wide as they get, then too many units
    (300_000, 128, 64, 10, 0.4), (65_664, 64, 200, 10, 0.9), (30_000, 700, 100, 20, 0.5),
])
def test_tied_rows_that_come_late(metric, n, d, nq, k, start):
    x, q = _codes(n, d, nq, n + k, 60)
    x -= 30.0
    x[int(start * n):] = 0.0 if metric == "l2sq" else 29.0
    q[:] = 0.0 if metric == "l2sq" else 20.0
    q[: nq // 2, 0] += 1.0
    _check_codes(x, q, k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
def test_tied_rows_behind_the_last_stage_only(metric):
    x, q = _codes(49_970, 64, 10, 3, 3)
    tail = 49_970 // 128 * 128
    assert tail < 49_970
    x[tail:] = 9.0
    x[tail + 7::2, 1] = 8.0
    q[:] = 9.0
    _check_codes(x, q, 20, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
def test_many_groups_above_the_bound(metric):
    """The nearest rows all in groups of nine of the sets that the bound, the tenth of the sets' maxima, is taken from: 144 groups
    lie above it and all others, whose rows are equal, at it."""
    n, d, nq, k = 150_077, 64, 300, 10
    G, S, SEG, waves, _, threads, _, _ = lpq.search_maxima_info(d, 8, False, n, nq, k)
    parts = 2 * waves
    assert waves == 4 and threads == 256 and 3072 < G <= 4096              # 256 sets of up to 16 groups
    x, q = _codes(n, d, nq, 11, 20)
    x[:] = 3.0
    row = torch.arange(n // 128 * 128, device="cuda")
    stage, part = row // 128, row % 128 // 32 * 2 + row % 8 // 4
    s, t = stage % S, stage // S
    T = (n // 128 - s + S - 1) // S
    group = (s * SEG + t * SEG // T) * parts + part
    near = row[group // 4 % 256 < 9]
    assert group[near].unique().numel() > 4 * k + 64
    g = torch.Generator(device="cuda").manual_seed(12)
    x[near] = 40.0 + torch.randint(0, 20, (near.numel(), d), generator=g, device="cuda").float()
    q += 40.0
    _check_codes(x, q, k, metric)
