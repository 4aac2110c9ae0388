"""The kernels that append candidates to a buffer in LDS step by step decide at each step, in all threads alike, whether it is
compacted.  With one counter for all steps a wave that was late read what faster ones had appended in the next step, went
the other way, and a query in some thousands lost neighbours: the same search again and again, against the oracle and
against slices.  Needs a real MI355X."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# k beyond what the matrix-core scans take; few and many features
@pytest.mark.parametrize("n,d,nq,k,metric", [(36_138, 11, 2499, 729, "ip"), (20_000, 300, 400, 1000, "l2sq")])
def test_generic_search_again_and_again(oracle, n, d, nq, k, metric):
    from paper_2110_08919_amd import lpq
    g = torch.Generator(device="cuda").manual_seed(d)
    x, q = torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")
    quant = lpq.Quantizer(d, 4).calibrate(x, "absmax", "global")
    index = lpq.Index(quant, n).add_f32(x)
    assert lpq.search_plan_info(d, 4, False, n, nq, k)[0] == 0
    oq = oracle.Quantizer(d, 4).set_params(*quant.get_params()[:3])
    ids, dists = oracle.search_i8(oq.encode(x.cpu().numpy()), oq.encode(q.cpu().numpy()), k, metric, threads=16)
    ids, dists = torch.from_numpy(np.asarray(ids)).cuda(), torch.from_numpy(np.asarray(dists)).cuda()
    for _ in range(30):
        got, gd = index.search(q, k, metric)
        assert torch.equal(got, ids) and torch.equal(gd, dists)


@pytest.mark.parametrize("n,d,nq,k", [(60_000, 6, 1500, 700), (60_000, 40, 3, 900)])
def test_direct_fp32_search_again_and_again(n, d, nq, k):
    from paper_2110_08919_amd import lpq
    from test_gpu_f32_filter import _direct, _same_bits
    import f32_plan
    g = torch.Generator(device="cuda").manual_seed(d)
    x, q = torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")
    assert not f32_plan.plan(n, nq, d, k)["use"]
    want = _direct(lpq, x, q, k, "l2sq")
    for _ in range(30):
        _same_bits(lpq.search_f32(x, q, k, "l2sq"), want)
