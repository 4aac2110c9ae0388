"""The matrix-core filter of the exact fp32 search: it must return, bit for bit, what the direct kernel
returns for the same queries on slices of the corpus too small for the filter, merged, and agree with
the CPU oracle.  Needs a real MI355X, but for the check of the compiled instruction order."""
import os
import re

import numpy as np
import pytest
import torch

from paper_2110_08919_amd import build as lpq_build, synth
from test_kernel_schedule import NEED, _closest_reads


def test_no_read_of_a_matrix_result_sooner_than_the_wait_states_it_needs():
    lpq_build.build()
    bad = _closest_reads(lpq_build.device_asm(os.path.join(lpq_build.CSRC, "search_mfma_f32.hip")))
    assert not bad, f"{len(bad)} reads of matrix results within {NEED} issue slots, e.g. {sorted(bad, key=lambda b: b[1])[:3]}"


def test_nothing_is_kept_in_scratch():
    """A reload from scratch waits for all loads of the stages on their way."""
    lpq_build.build()
    asm = open(lpq_build.device_asm(os.path.join(lpq_build.CSRC, "search_mfma_f32.hip"))).read()
    spills = dict(re.findall(r"\.name: +(\S*filter_f32_kernel\S*)\n(?:.*\n)*?.*\.vgpr_spill_count: (\d+)", asm))
    assert len(spills) == 18 and not any(map(int, spills.values())), spills


@pytest.fixture(scope="module")
def lpq():
    from paper_2110_08919_amd import lpq as m
    assert torch.cuda.is_available(), "no GPU visible"
    m.lib()
    return m


def _direct(lpq, x, q, k, metric):
    """Direct kernel on slices of 4000 rows (the filter starts at 4096), merged by (distance, id).
    Values are ranked the way the kernels rank them: by an order-preserving integer image."""
    ids, keys, dists = [], [], []
    for r0 in range(0, x.shape[0], 4000):
        part = x[r0:r0 + 4000]
        i, v = lpq.search_f32(part, q, min(k, part.shape[0]), metric)
        b = (v if metric == "l2sq" else -v).add(0.0).view(torch.int32)
        ids.append(i.long() + r0)
        keys.append(torch.where(b >= 0, b, b ^ 0x7FFFFFFF).long())
        dists.append(v)
    ids, keys, dists = torch.cat(ids, 1), torch.cat(keys, 1), torch.cat(dists, 1)
    order = ((keys << 32) + ids).argsort(dim=1)[:, :k]
    return ids.gather(1, order).int(), dists.gather(1, order)


def _same_bits(got, want):
    torch.cuda.synchronize()
    assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
    assert torch.equal(got[0], want[0])


# both query tiles, features that end inside a stage and inside a 16-byte load, rows that end inside a tile
@pytest.mark.gpu
@pytest.mark.parametrize("recipe,n,d,nq,k,metric", [
    ("bimodal", 20_000, 128, 300, 10, "l2sq"),
    ("scaled_unit", 16_385, 24, 64, 1, "ip"),
    ("bimodal", 50_000, 96, 1, 10, "l2sq"),
    ("scaled_unit", 5000, 24, 16_500, 2, "l2sq"),        # two batches of queries
    ("bimodal", 300_000, 40, 3000, 10, "ip"),            # one or two splits of the corpus per query tile
    ("scaled_unit", 30_001, 33, 65, 100, "l2sq"),
    ("skewed_int", 40_000, 100, 500, 10, "l2sq"),        # integer data: many equal distances
    ("skewed_int", 25_000, 31, 129, 20, "ip"),
    ("bimodal", 12_345, 515, 80, 33, "ip"),
    ("scaled_unit", 9000, 1024, 100, 7, "l2sq"),
])
def test_filtered_search_returns_the_direct_kernels_bits(lpq, oracle, recipe, n, d, nq, k, metric):
    w = synth.Workload("w", recipe, n, d, nq, metric, (k,), "minmax", "global", 9)
    x, q = w.corpus("cuda"), w.queries("cuda")
    got = lpq.search_f32(x, q, k, metric)
    _same_bits(got, _direct(lpq, x, q, k, metric))
    sub = slice(0, 20)
    _, od = oracle.search_f32(x.cpu().numpy(), q.cpu().numpy()[sub], k, metric, threads=16)
    # relative to the value, or for inner products that cancel to |q||x|
    floor = 0.0 if metric == "l2sq" else float(torch.linalg.vector_norm(x, dim=1).max() * torch.linalg.vector_norm(q, dim=1).max())
    assert np.all(np.abs(got[1].cpu().numpy()[sub] - od) <= 1e-5 * np.maximum(np.abs(od), floor))


@pytest.mark.gpu
def test_filtered_search_takes_strided_and_unaligned_rows(lpq):
    w = synth.Workload("w", "bimodal", 15_000, 101, 90, "l2sq", (10,), "minmax", "global", 2)
    x, q = w.corpus("cuda"), w.queries("cuda")
    want = _direct(lpq, x[:, 1:100].contiguous(), q[:, 1:100].contiguous(), 10, "l2sq")
    _same_bits(lpq.search_f32(x[:, 1:100], q[:, 1:100], 10, "l2sq"), want)


@pytest.mark.gpu
@pytest.mark.parametrize("metric", ["l2sq", "ip"])
def test_filtered_search_of_data_the_bounds_do_not_resolve(lpq, metric):
    """Distances tiny next to the norms (everything passes the filter), values whose squares overflow or
    underflow, infinities and NaN: those queries go through the direct kernel."""
    g = torch.Generator(device="cuda").manual_seed(3)
    n, d, nq, k = 10_000, 40, 100, 10
    x, q = torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")
    for scale, shift in ((1.0, 3000.0), (1e17, 0.0), (1e-25, 0.0), (0.0, 1.0)):
        xs, qs = x * scale + shift, q * scale + shift
        _same_bits(lpq.search_f32(xs, qs, k, metric), _direct(lpq, xs, qs, k, metric))
    for value in (float("inf"), float("nan"), 3e38):
        xs, qs = x.clone(), q.clone()
        xs[4321, 7] = value                     # one bad row
        _same_bits(lpq.search_f32(xs, qs, k, metric), _direct(lpq, xs, qs, k, metric))
        qs[50, 3] = value                       # a bad query beside good ones
        _same_bits(lpq.search_f32(x, qs, k, metric), _direct(lpq, x, qs, k, metric))


@pytest.mark.gpu
def test_filtered_search_of_clustered_and_duplicated_rows(lpq):
    g = torch.Generator(device="cuda").manual_seed(5)
    n, d, nq, k = 20_000, 64, 200, 20
    centres = torch.randn((20, d), generator=g, device="cuda")
    x = centres.repeat_interleave(n // 20, 0) + 0.05 * torch.randn((n, d), generator=g, device="cuda")
    x[10_000:15_000] = x[5000:10_000]
    q = torch.cat([x[4990:5090], centres.repeat(5, 1)])
    for metric in ("l2sq", "ip"):
        _same_bits(lpq.search_f32(x, q, k, metric), _direct(lpq, x, q, k, metric))
