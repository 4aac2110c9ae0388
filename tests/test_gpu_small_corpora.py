"""Small corpora cut into splits of 128 rows, and the merge of many sorted lists: bit-exact against the
CPU oracle.  Needs a real MI355X."""
import numpy as np
import pytest
import torch

from paper_2110_08919_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lpq():
    from paper_2110_08919_amd import lpq as m
    assert torch.cuda.is_available(), "no GPU visible"
    m.lib()
    return m


# lists per query on both sides of 26 (a plain sort below), 256 and 512 (lists per thread), k on both
# sides of 16 (two sizes of the bound's sort) and at 32; few and many queries; corpora just above 4096 rows
@pytest.mark.parametrize("n,d,nq,k,metric,bits", [
    (4099, 128, 1, 10, "l2sq", 8), (4200, 64, 300, 3, "ip", 8), (10_000, 128, 100, 10, "l2sq", 8),
    (20_001, 96, 64, 10, "l2sq", 8), (33_000, 128, 16, 1, "ip", 8), (40_000, 128, 65, 16, "l2sq", 8),
    (66_000, 100, 64, 10, "ip", 8), (70_000, 64, 5, 10, "l2sq", 1), (36_000, 128, 8, 16, "ip", 1),
    (150_000, 96, 2, 10, "l2sq", 8), (9000, 300, 1000, 10, "l2sq", 8),
])
def test_small_corpus_search(lpq, oracle, n, d, nq, k, metric, bits):
    w = synth.Workload("w", "skewed_int", n, d, nq, metric, (k,), "minmax", "global", 4)
    x, q = w.corpus("cuda"), w.queries("cuda")
    gq = lpq.Quantizer(d, bits).calibrate(x, "minmax" if metric == "l2sq" else "absmax", "global")
    ids, dists = lpq.Index(gq, n).add_f32(x).search(q, k, metric)
    kk, sb, se, _ = gq.get_params()
    oq = oracle.Quantizer(d, bits).set_params(kk, sb, se)
    oids, odists = oracle.search_i8(oq.encode(x.cpu().numpy()), oq.encode(q.cpu().numpy()), k, metric, threads=16)
    assert np.array_equal(dists.cpu().numpy(), odists) and np.array_equal(ids.cpu().numpy(), oids)


@pytest.mark.parametrize("n,k", [(3000, 10), (4000, 20), (4000, 32)])
def test_merge_of_sorted_lists_with_few_candidates(lpq, n, k):
    """The direct fp32 kernel's lists: k up to 32 from one or two splits, equal distances everywhere."""
    x = torch.zeros((n, 20), device="cuda")
    x[: n // 2] = 1.0
    ids, dists = lpq.search_f32(x, x[:3], k, "l2sq")
    assert torch.equal(ids.cpu(), torch.arange(k, dtype=torch.int32).expand(3, k)) and not dists.any()


@pytest.mark.parametrize("n,d,nq,k", [(100_000, 256, 256, 10), (10_000, 32, 2000, 10), (5000, 2048, 3000, 10), (50_000, 100, 700, 100)])
def test_static_search_of_shapes_whose_normal_plan_needs_more(lpq, n, d, nq, k):
    """The library's own workspace of 64 MiB: a search whose plan does not fit takes one that does."""
    w = synth.Workload("w", "bimodal", n, d, nq, "l2sq", (k,), "minmax", "global", 7)
    x, q = w.corpus("cuda"), w.queries("cuda")
    index = lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "minmax", "global"), n).add_f32(x)
    assert index.workspace_bytes(nq, k) > lpq.STATIC_WORKSPACE_BYTES
    want, got = index.search(q, k), index.search_static(q, k)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
