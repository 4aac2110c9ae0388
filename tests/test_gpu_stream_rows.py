"""The scan that streams both operands (rows of more than 1536 features), bit-exact on ids and int32
distances against the CPU oracle, or against the generic dot-product kernel where the oracle would
take too long.  Needs a real MI355X, but for the check of the compiled instruction order."""
import os

import numpy as np
import pytest
import torch

from paper_2110_08919_amd import build as lpq_build, synth
from test_kernel_schedule import NEED, _closest_reads


def test_no_read_of_a_matrix_result_sooner_than_the_wait_states_it_needs():
    lpq_build.build()
    path = lpq_build.device_asm(os.path.join(lpq_build.CSRC, "search_mfma_stream.hip"))
    assert os.path.exists(path)
    bad = _closest_reads(path)
    assert not bad, f"{len(bad)} reads of matrix results within {NEED} issue slots, e.g. {sorted(bad, key=lambda b: b[1])[:3]}"


@pytest.fixture(scope="module")
def lpq():
    from paper_2110_08919_amd import lpq as m
    assert torch.cuda.is_available(), "no GPU visible"
    m.lib()
    return m


def _generic(lpq, index, q, k, metric):
    lpq.set_tuning(lpq.TUNE_PATH, 1)
    try:
        ids, dists = index.search(q, k, metric)
        torch.cuda.synchronize()
    finally:
        lpq.set_tuning(lpq.TUNE_PATH, 0)
    return ids, dists


def _same(got, want):
    torch.cuda.synchronize()
    assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0])


# query tiles of 64, 128 and 256 (both sides of each limit), rows that end inside a stage, corpora that
# end inside a tile, one tile per split and many
@pytest.mark.gpu
@pytest.mark.parametrize("recipe,d,n,nq,k,metric", [
    ("bimodal", 1537, 20_003, 1, 10, "l2sq"),
    ("bimodal", 1600, 20_000, 64, 1, "ip"),
    ("skewed_int", 1601, 33_025, 65, 100, "l2sq"),
    ("bimodal", 2048, 16_384, 128, 17, "l2sq"),
    ("scaled_unit", 2047, 16_641, 129, 10, "ip"),
    ("bimodal", 3000, 12_000, 300, 33, "l2sq"),
    ("scaled_unit", 4096, 9_000, 257, 3, "ip"),
])
def test_search_streamed_rows(lpq, oracle, recipe, d, n, nq, k, metric):
    assert lpq.search_plan_info(d, 8, 0, n, nq, k)[0] == 3, "the collecting scan was expected here"
    w = synth.Workload("w", recipe, n, d, nq, metric, (k,), "minmax", "global", 5)
    x, q = w.corpus("cuda"), w.queries("cuda")
    gq = lpq.Quantizer(d, 8).calibrate(x, "minmax" if metric == "l2sq" else "absmax", "per_feature")
    index = lpq.Index(gq, n).add_f32(x)
    got = index.search(q, k, metric)
    kk, sb, se, _ = gq.get_params()
    oq = oracle.Quantizer(d, 8).set_params(kk, sb, se)
    oids, odists = oracle.search_i8(oq.encode(x.cpu().numpy()), oq.encode(q.cpu().numpy()), k, metric, threads=16)
    assert np.array_equal(got[1].cpu().numpy(), odists) and np.array_equal(got[0].cpu().numpy(), oids)
    _same(index.search(gq.encode(q), k, metric), got)      # queries that are codes already


@pytest.mark.gpu
@pytest.mark.parametrize("d,nq,k", [(1700, 700, 100), (2048, 100, 20), (2500, 40, 128)])
def test_search_streamed_rows_overflow_is_redone_exactly(lpq, d, nq, k):
    """Regions of two candidates: every query goes through the further rounds and the generic kernel."""
    w = synth.Workload("w", "skewed_int", 20_000, d, nq, "l2sq", (k,), "minmax", "global", 6)
    x, q = w.corpus("cuda"), w.queries("cuda")
    index = lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "minmax", "global"), 20_000).add_f32(x)
    want = _generic(lpq, index, q, k, "l2sq")
    lpq.set_tuning(lpq.TUNE_REGION_CAP, 2)
    try:
        _same(index.search(q, k, "l2sq"), want)
    finally:
        lpq.set_tuning(lpq.TUNE_REGION_CAP, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [1537, 32_768])
def test_search_streamed_rows_extreme_codes_and_duplicates(lpq, d):
    """Codes at the ends of the range (the largest products and norms an int32 must hold), every item
    present twice: ties go to the lower id."""
    n, nq, k = 5000, 70, 12
    r = np.random.default_rng(8)
    c = r.choice(np.array([-128, 127], np.int8), size=(n // 2, d))
    c = torch.as_tensor(np.concatenate([c, c])).cuda()
    q = torch.cat([c[:35], torch.as_tensor(r.choice(np.array([-128, 127], np.int8), size=(35, d))).cuda()])
    gq = lpq.Quantizer(d, 8).set_params(np.zeros(d), np.full(d, -128.0), np.full(d, 128.0))
    index = lpq.Index(gq, n + 300).add_i8(c)      # room for more rows than there are
    for metric in ("l2sq", "ip"):
        got = index.search(q, k, metric)
        _same(got, _generic(lpq, index, q, k, metric))
    ids, dists = index.search(q, 2, "l2sq")
    assert torch.equal(ids[:35, 0].cpu(), torch.arange(35, dtype=torch.int32)) and not dists[:35].any()
    assert torch.equal(ids[:35, 1].cpu(), torch.arange(35, dtype=torch.int32) + n // 2)


@pytest.mark.gpu
def test_search_streamed_rows_corpus_sorted_by_cluster(lpq):
    """Near neighbours in adjacent rows: the sample is spread over the corpus and the result exact."""
    d, n, nq, k = 1600, 30_000, 200, 20
    g = torch.Generator(device="cuda").manual_seed(4)
    centres = torch.randint(-100, 100, (30, d), generator=g, device="cuda")
    x = (centres.repeat_interleave(n // 30, 0) + torch.randint(-9, 10, (n, d), generator=g, device="cuda")).to(torch.int8)
    q = (centres[torch.randint(0, 30, (nq,), generator=g, device="cuda")]
         + torch.randint(-9, 10, (nq, d), generator=g, device="cuda")).to(torch.int8)
    gq = lpq.Quantizer(d, 8).set_params(np.zeros(d), np.full(d, -128.0), np.full(d, 128.0))
    index = lpq.Index(gq, n).add_i8(x)
    for metric in ("l2sq", "ip"):
        _same(index.search(q, k, metric), _generic(lpq, index, q, k, metric))


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,nq,k", [(32, 3511, 17_478, 10), (3, 4248, 15_190, 3), (3000, 1805, 5041, 700)])
def test_static_search_of_batches_that_row_padding_pushes_over_the_limit(lpq, n, d, nq, k):
    """The codes of these queries fit the built-in workspace with rows padded to 32 bytes, but not to 128."""
    w = synth.Workload("w", "bimodal", n, d, nq, "l2sq", (k,), "minmax", "global", 7)
    x, q = w.corpus("cuda"), w.queries("cuda")
    index = lpq.Index(lpq.Quantizer(d, 8).calibrate(x, "minmax", "global"), n).add_f32(x)
    want, got = index.search(q, k), index.search_static(q, k)
    _same(got, want)
