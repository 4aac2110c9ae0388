"""Queries whose nearest items all lie in the sample of the collecting scan: its bound, the rank-th largest maximum of the
sample, lets fewer than k items pass, which is found by their count and searched again.  One, some and many such queries
for each of the scans, against the generic kernel.  Needs a real MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _shift(unit, room):
    return (((unit * 0x9E3779B1) & 0xFFFFFFFF) * (room + 1)) >> 32


def _sampled_rows(n, d, nq, plan):
    """A row of each run or stage of the sample, neighbours in different groups of the pass."""
    seed_rows, splits = plan[5], plan[6]
    if d > 512:      # tiles of sixteen runs of 16 rows
        tiles = seed_rows // 256
        stride = n // (16 * tiles)
        return [(i * tiles + g) * stride + _shift(g, stride - 16) for i in range(16) for g in range(tiles)]
    if d > 256:      # stages of 32 or 64 rows
        rows = 64 if nq > 512 else 32
        stages = seed_rows // (rows * splits)
        stride = n // (stages * splits) // 128 * 128
        return [(s * stages + t) * stride + _shift(s + splits * t, stride - rows) for t in range(stages) for s in range(splits)]
    stages = seed_rows // (64 * splits)
    stride = n // (8 * stages * splits)
    return [(s + splits * (8 * t + p)) * stride + _shift(s + splits * t, stride - 8)
            for t in range(stages) for p in range(8) for s in range(splits)]


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k,short", [
    (200_000, 64, 300, 16, 1), (200_000, 128, 2000, 16, 70),     # by the generic kernel, by the register lists
    (200_000, 100, 300, 60, 2), (300_000, 128, 2100, 30, 40),    # by the generic kernel at once, by a further round
    (200_000, 384, 600, 30, 15), (100_000, 700, 600, 20, 9),     # long rows, streamed rows (more than 512 queries: smaller batches are not sampled)
])
def test_queries_with_too_few_candidates(metric, n, d, nq, k, short):
    from paper_2110_08919_amd import lpq
    g = torch.Generator(device="cuda").manual_seed(n + d)
    x, q = ((torch.randn((m, d), generator=g, device="cuda") * 10).round_().clamp_(-60, 60) for m in (n, nq))
    plan = lpq.search_plan_info(d, 8, False, n, nq, k)
    assert plan[0] == 3 and plan[5] > 0
    rows = _sampled_rows(n, d, nq, plan)
    assert len(rows) >= short * k and max(rows) < n
    for j in range(short):
        for i in range(k):                       # the k nearest of query j, no two at the same distance
            x[rows[j * k + i]] = q[j]
            x[rows[j * k + i], i % d] += i + 1
    quant = lpq.Quantizer(d, 8)
    quant.set_params([0.0] * d, [-128.0] * d, [128.0] * d)
    index = lpq.Index(quant, n).add_f32(x)
    ids, dists = index.search(q, k, metric)
    torch.cuda.synchronize()
    assert index.overflow_stats(nq, k, metric)[0] >= short
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q, k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists, want) and torch.equal(ids, want_ids)
