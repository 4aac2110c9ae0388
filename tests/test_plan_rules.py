"""Which scan a search takes and how much workspace it asks for (computed on the host, no GPU needed)."""
import numpy as np
import pytest
import torch

from paper_2110_08919_amd import lpq, synth

REGISTER_LISTS, COLLECTING = 2, 3


def _plan(d, bits, n, nq, k):
    """(mode, workspace in MB) of a flat index' search."""
    p = lpq.search_plan_info(d, bits, False, n, nq, k)
    return p[0], p[16] >> 20


# Many items tie on codes of one bit (on two, in larger corpora), and all that tie at the bound is collected.
@pytest.mark.parametrize("bits,n", [(1, 5000), (1, 20_000), (1, 1_000_000), (1, 4_000_000), (2, 32_769), (2, 1_000_000)])
@pytest.mark.parametrize("nq", [65, 100, 256, 513, 700, 768])
def test_codes_of_few_bits_keep_the_register_lists(bits, n, nq):
    for k in (1, 10):
        mode, mb = _plan(128, bits, n, nq, k)
        assert mode == REGISTER_LISTS and mb <= 40


@pytest.mark.parametrize("nq", [300, 1000, 10_000])
def test_one_bit_codes_keep_the_register_lists_at_every_batch_size(nq):
    for n in (20_000, 1_000_000):
        mode, mb = _plan(128, 1, n, nq, 10)
        assert mode == REGISTER_LISTS and mb <= 40


@pytest.mark.parametrize("bits,n,nq,k,mode", [
    (8, 5000, 65, 5, COLLECTING), (8, 5000, 65, 4, REGISTER_LISTS), (8, 20_000, 256, 10, COLLECTING),
    (8, 50_000, 100, 10, COLLECTING), (8, 50_001, 100, 10, REGISTER_LISTS), (3, 300_000, 640, 10, COLLECTING),
    (2, 32_768, 100, 10, COLLECTING), (8, 1_000_000, 100, 10, REGISTER_LISTS), (8, 1_000_000, 640, 10, REGISTER_LISTS),
    (8, 1_000_000, 300, 10, COLLECTING), (8, 1_000_000, 1000, 10, COLLECTING), (8, 1_000_000, 100, 11, COLLECTING),
])
def test_small_batches_collect_on_small_corpora_only(bits, n, nq, k, mode):
    assert _plan(128, bits, n, nq, k)[0] == mode


@pytest.mark.parametrize("d", [513, 1024, 2048, 4096])
@pytest.mark.parametrize("n", [4096, 4097, 8000, 10_000, 20_000, 60_001])
def test_streamed_rows_have_a_tile_for_every_split(d, n):
    """Splits and regions (7 and 10 of the plan) that no tile of 256 rows falls to."""
    for nq in (1, 64, 100, 300, 1000, 10_000):
        for k in (1, 10, 30):
            p = lpq.search_plan_info(d, 8, False, n, nq, k)
            assert p[0] != COLLECTING or (p[7] <= -(-n // 256) and p[10] == p[7])


@pytest.mark.gpu
@pytest.mark.parametrize("bits,n,nq,k,calib,scope", [
    (1, 40_000, 300, 10, "minmax", "per_feature"), (1, 40_000, 700, 10, "absmax", "global"),
    (2, 40_000, 200, 10, "minmax", "global"), (2, 20_000, 600, 7, "minmax", "global"), (8, 60_000, 128, 10, "minmax", "global"),
])
def test_search_on_both_sides_of_the_rule(oracle, bits, n, nq, k, calib, scope):
    w = synth.Workload("w", "skewed_int", n, 128, nq, "l2sq", (k,), calib, scope, 4)
    x, q = w.corpus("cuda"), w.queries("cuda")
    gq = lpq.Quantizer(128, bits).calibrate(x, calib, scope)
    ids, dists = lpq.Index(gq, n).add_f32(x).search(q, k)
    kk, sb, se, _ = gq.get_params()
    oq = oracle.Quantizer(128, bits).set_params(kk, sb, se)
    oids, odists = oracle.search_i8(oq.encode(x.cpu().numpy()), oq.encode(q.cpu().numpy()), k, "l2sq", threads=16)
    assert np.array_equal(dists.cpu().numpy(), odists) and np.array_equal(ids.cpu().numpy(), oids)
