"""Selection among collected candidates for k beyond 16, where ranks are counted: few candidates, one more than the kernel
holds at a time, and keys of so few values that the last bin of its histogram holds more than it counts ranks for.
Against the generic kernel.  Needs a real MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k,levels,seed_rows", [
    (100_000, 64, 300, 17, 0, 0),
    (100_000, 64, 70, 100, 0, 4096),        # some 2500 candidates a query
    (150_000, 96, 80, 128, 0, 16_384),      # ... about 1200
    (60_000, 8, 200, 64, 3, 0),             # three values per feature: distances tie by the hundreds
    (100_000, 32, 1500, 33, 5, 8192),
])
def test_selected_candidates(metric, n, d, nq, k, levels, seed_rows):
    from paper_2110_08919_amd import lpq
    g = torch.Generator(device="cuda").manual_seed(k)
    if levels:
        x, q = (torch.randint(0, levels, (m, d), generator=g, device="cuda").float() for m in (n, nq))
    else:
        x, q = (torch.randn((m, d), generator=g, device="cuda") for m in (n, nq))
    quant = lpq.Quantizer(d, 8).calibrate(x, "absmax", "global")
    index = lpq.Index(quant, n).add_f32(x)
    lpq.set_tuning(lpq.TUNE_SEED_ROWS, seed_rows)
    try:
        ids, dists = index.search(q, k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_SEED_ROWS, 0)
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q, k, metric)
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists, want) and torch.equal(ids, want_ids)


# large batches leave few regions per query, whose candidates the lanes of a workgroup share: 1, 2, 5 and 12 regions
@pytest.mark.parametrize("n,d,nq,k,regions", [(40_000, 32, 150_000, 100, 1), (60_000, 32, 130_000, 17, 2), (100_000, 32, 50_000, 100, 5),
                                              (100_000, 64, 20_000, 64, 12)])
def test_candidates_of_few_regions(n, d, nq, k, regions):
    from paper_2110_08919_amd import lpq
    g = torch.Generator(device="cuda").manual_seed(nq)
    x, q = (torch.randn((m, d), generator=g, device="cuda") for m in (n, nq))
    quant = lpq.Quantizer(d, 8).calibrate(x, "absmax", "global")
    index = lpq.Index(quant, n).add_f32(x)
    assert lpq.search_plan_info(d, 8, False, n, nq, k)[7] == regions
    ids, dists = index.search(q, k, "l2sq")
    sub = torch.cat([torch.arange(300), torch.arange(nq - 300, nq)]).cuda()
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        want_ids, want = index.search(q[sub].contiguous(), k, "l2sq")
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    torch.cuda.synchronize()
    assert torch.equal(dists[sub], want) and torch.equal(ids[sub], want_ids)
