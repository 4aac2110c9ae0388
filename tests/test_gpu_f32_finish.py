"""The end of the fp32 search: of the rows its filter collected only those whose upper bounds still matter are summed
directly.  Same bits as the direct kernel alone; from a handful of candidates per query to more than the workgroup holds
at a time.  Needs a real MI355X."""
import pytest
import torch

from test_gpu_f32_filter import _direct, _same_bits

pytestmark = pytest.mark.gpu


def _check(x, q, k, metric):
    from paper_2110_08919_amd import lpq
    _same_bits(lpq.search_f32(x, q, k, metric), _direct(lpq, x, q, k, metric))


# k below and above what is summed first at least, ranks counted and sorted (beyond 512), candidates beyond 2048
@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(5000, 8, 300, 1), (5000, 7, 65, 39), (60_000, 33, 40, 300), (200_000, 16, 40, 480), (70_000, 130, 20, 512)])
def test_candidates_of_any_number(metric, n, d, nq, k):
    g = torch.Generator(device="cuda").manual_seed(k)
    x, q = torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")
    q[0] *= 1e-3                               # scores of both signs next to zero
    _check(x, q, k, metric)


# the spread decides how many rows lie within the bounds' error of the nearest: hundreds to more than regions hold
@pytest.mark.parametrize("spread", [0.45, 0.55, 0.65, 0.8, 1.2])
def test_rows_within_the_error_of_the_bounds(spread):
    g = torch.Generator(device="cuda").manual_seed(9)
    x, q = torch.randn((200_000, 16), generator=g, device="cuda"), torch.randn((40, 16), generator=g, device="cuda")
    _check(spread * x + 20.0, spread * q + 20.0, 10, "l2sq")


def test_equal_distances():
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randint(0, 3, (30_000, 9), generator=g, device="cuda").float()
    q = torch.randint(0, 3, (100, 9), generator=g, device="cuda").float()
    for metric in ("l2sq", "ip"):
        _check(x, q, 10, metric)


# bounds of the first scan, scaled by the powers of two of rows and queries, of shifted data: more candidates than are kept in
# LDS (2048), more than 512 rows to rank, and a few
@pytest.mark.parametrize("metric,k,shift,scale,least", [("l2sq", 400, 4.0, 1e-6, 2500), ("l2sq", 500, 4.0, 300.0, 3000), ("ip", 500, 15.0, 1e-6, 2600),
                                                        ("ip", 500, 15.0, 1e4, 2600), ("l2sq", 10, 2.0, 1e-6, 150), ("ip", 10, 15.0, 1.0, 150)])
def test_candidates_of_the_first_scan(metric, k, shift, scale, least):
    import f32_plan
    from paper_2110_08919_amd import lpq
    g = torch.Generator(device="cuda").manual_seed(1)
    x, q = torch.randn((200_000, 64), generator=g, device="cuda"), torch.randn((400, 64), generator=g, device="cuda")
    x, q = scale * (x + shift), scale * (q + shift)
    got, p, ws = f32_plan.search(x, q, k, metric)
    _same_bits(got, _direct(lpq, x, q, k, metric))
    counts = f32_plan.words(p, ws, "off_ccnt", 400 * p["S2"]).view(400, -1).sum(1)
    again, hard, over = (f32_plan.words(p, ws, name, m) for name, m in (("off_again", 400), ("off_hard", 4), ("off_over", 400)))
    assert p["half"] and not bool(again.any() or hard.any() or over.any()) and int(counts.max()) >= least


def test_giving_up_on_candidates_costs_a_fraction_of_the_direct_kernel():
    """Some 10 000 rows of a query within the error of their bounds, in regions that hold them.  With all of them sorted
    the search took 1.7 times as long as the direct kernel alone."""
    from paper_2110_08919_amd import lpq
    from f32_plan import best_ms
    g = torch.Generator(device="cuda").manual_seed(2)
    x, q = torch.randn((1_000_000, 128), generator=g, device="cuda"), torch.randn((1, 128), generator=g, device="cuda")
    x[::100] *= 1e4
    bad = x.clone()
    bad[:, 0] = float("nan")               # to the direct kernel, nothing collected
    assert best_ms(lambda: lpq.search_f32(x, q, 10, "ip")) <= 1.35 * best_ms(lambda: lpq.search_f32(bad, q, 10, "ip"))
