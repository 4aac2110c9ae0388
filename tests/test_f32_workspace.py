"""Workspace of the exact fp32 search: large batches are searched in parts; rows too far apart for its filter's offsets.
The sizes need no GPU."""
import subprocess

import pytest
import torch

from paper_2110_08919_amd import build as lpq_build
from paper_2110_08919_amd import lpq, synth


@pytest.mark.parametrize("n", [5000, 60_000, 447_990, 1_000_000, 50_000_000])
@pytest.mark.parametrize("d", [16, 128, 771])
def test_workspace_is_bounded_for_any_batch_and_k(n, d):
    for k in (1, 10, 100, 480, 505, 1024):
        for nq in (256, 257, 1000, 8192, 10_000, 16_384, 16_385, 20_580, 100_000, 1_000_000):
            # 256 MB and the rounding of the query
            assert 0 < lpq.lib().lpq_search_f32_workspace_bytes(n, nq, d, k) <= (256 << 20) + 256


def test_rows_of_a_tile_lie_within_32_bit_offsets(tmp_path):
    """Rows any further apart (4096 of them span 276 GB) are left to the direct kernel, whose offsets have 64 bits."""
    src, exe = tmp_path / "c.hip", str(tmp_path / "c")
    src.write_text('#include <cstdio>\n#include "lpq_internal.h"\n'
                   'int main() { for (int d : {1, 4, 128, 16384}) std::printf("%d %lld\\n", d, (long long)lpq::f32_filter_max_ld(d)); }\n')
    subprocess.run([lpq_build.HIPCC, *lpq_build.FLAGS, str(src), "-o", exe], check=True)
    for line in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines():
        d, ld = map(int, line.split())
        last = 255 * ld + d - 1                      # last value of a tile's last row
        assert last < 2 ** 32 <= last + 255 + d


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,nq,k", [(30_000, 16, 15_001, 100)])
def test_search_in_parts_equals_the_same_queries_searched_apart(n, d, nq, k):
    w = synth.Workload("w", "bimodal", n, d, nq, "l2sq", (k,), "minmax", "global", 3)
    x, q = w.corpus("cuda"), w.queries("cuda")
    ids, dists = lpq.search_f32(x, q, k, "l2sq")
    for q0, q1 in ((0, 70), (nq // 2 - 40, nq // 2 + 40), (nq - 50, nq)):
        i, v = lpq.search_f32(x, q[q0:q1], k, "l2sq")
        torch.cuda.synchronize()
        assert torch.equal(ids[q0:q1], i) and torch.equal(dists[q0:q1], v)


def test_regions_have_room_for_uneven_filling():
    """Regions of the fp32 filter that a query is expected to fill by more than half hold 128 candidates, not 64."""
    import f32_plan
    assert f32_plan.plan(1_357_103, 9019, 37, 2)["Cs"] == 128
    assert f32_plan.plan(1_000_000, 1000, 128, 10)["Cs"] == 64
