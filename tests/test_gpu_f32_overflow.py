"""The fp32 search's filter on data it cannot filter: a query whose region overflows is given up, a workgroup
with none left ends early, and the direct kernel answers.  Same bits as the direct kernel alone.
Needs a real MI355X."""
import pytest
import torch

import f32_plan
from paper_2110_08919_amd import lpq
from test_gpu_f32_filter import _direct, _same_bits

pytestmark = pytest.mark.gpu


def _data(n, d, nq, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")


# one stage to a tile and several, both query tiles, few and many tiles to a split
@pytest.mark.parametrize("n,d,nq", [(9000, 24, 64), (40_000, 40, 300), (60_000, 100, 4000), (150_000, 33, 200)])
def test_queries_that_overflow_beside_queries_that_do_not(n, d, nq):
    """Half of the corpus around a far centre, where the bounds resolve nothing: queries near it overflow,
    queries near the origin do not; all of one kind, and both in one tile."""
    k = 10
    x, q = _data(n, d, nq, 3)
    x[n // 2:] = 0.01 * x[n // 2:] + 3000.0
    far, row = 0.01 * q + 3000.0, torch.arange(nq, device="cuda")[:, None]
    for mix in (q, far, torch.where(row % 7 == 0, far, q), torch.where(row < nq // 2, far, q), torch.where(row == nq - 1, q, far)):
        _same_bits(lpq.search_f32(x, mix, k, "l2sq"), _direct(lpq, x, mix, k, "l2sq"))


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(9000, 24, 60, 10), (70_000, 33, 3000, 5)])
def test_rows_that_are_not_finite_or_huge(metric, n, d, nq, k):
    x, q = _data(n, d, nq, 1)
    for rows in ([n // 2], [0, n - 1], range(0, n, 50)):
        for value in (float("nan"), float("inf"), 3e38):
            xs = x.clone()
            xs[list(rows), n // 3 % d] = value
            _same_bits(lpq.search_f32(xs, q, k, metric), _direct(lpq, xs, q, k, metric))


def test_a_second_round_of_workgroups_leaves_out_what_the_first_has_given_up():
    """1000 queries take 512 workgroups, twice what the GPU holds at a time."""
    n, d, nq, k = 200_000, 64, 1000, 10
    x, q = _data(n, d, nq, 5)
    x, q = x + 3000.0, q + 3000.0
    got, p, ws = f32_plan.search(x, q, k, "l2sq")
    _same_bits(got, _direct(lpq, x, q, k, "l2sq"))
    assert p["half"] and p["qtiles"] * p["S2"] == 512
    given_up = f32_plan.words(p, ws, "off_ccnt", nq * p["S2"]) > p["Cs"]
    empty = f32_plan.words(p, ws, "off_cbuf", nq * p["S2"] * p["Cs"] * 2).view(-1, p["Cs"] * 2)[:, :2].eq(0).all(dim=1)
    assert bool(given_up.all()) and float(empty.float().mean()) > 0.25


def test_giving_up_costs_a_fraction_of_the_direct_kernel():
    """With every item queued it took 1.4 times as long; giving up takes 1.06, 1.11 as the first work of a process."""
    n, d, nq, k = 200_000, 64, 1000, 10
    x, q = _data(n, d, nq, 4)
    x, q = x + 3000.0, q + 3000.0

    def best(fn):
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fn()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    bad = x.clone()
    bad[:, 0] = float("nan")              # every query to the direct kernel, nothing collected
    assert best(lambda: lpq.search_f32(x, q, k, "l2sq")) <= 1.25 * best(lambda: lpq.search_f32(bad, q, k, "l2sq"))
