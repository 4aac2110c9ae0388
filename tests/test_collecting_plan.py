"""Sample and regions of the collecting scan (no device needed): a sample by the bound's rank lets no more candidates through than one of the
rule for the k-th largest maximum, and the regions hold what that lets through, three times."""
import math

import pytest

from paper_2110_08919_amd import lpq


@pytest.mark.parametrize("d,n,nq,k", [(107, 1_324_429, 2363, 10), (128, 1_000_000, 10_000, 10), (200, 500_000, 1000, 10), (64, 1_000_000, 3000, 10),
                                      (96, 4_000_000, 5000, 5), (187, 1_604_278, 558, 1)])
def test_small_k_keeps_a_large_sample(d, n, nq, k):
    rows = 125_000 * math.sqrt(n / 1e6 * k / 10)
    p = lpq.search_plan_info(d, 8, False, n, nq, k)
    assert p[0] == 3 and p[5] > 0.7 * rows            # (shares of the corpus are tried in steps of a seventh; fewer rows where the rank is below k)


@pytest.mark.parametrize("d,n,nq,k", [(74, 673_620, 8080, 200), (541, 79_076, 4465, 100), (281, 156_655, 6979, 200), (256, 4_000_000, 10_000, 100),
                                      (128, 1_000_000, 3000, 512), (128, 1_000_000, 10_000, 100), (768, 500_000, 10_000, 100)])
def test_regions_hold_the_candidates_of_the_rule_before(d, n, nq, k):
    rows = 125_000 * math.sqrt(n / 1e6 * k / 10) * (math.sqrt(128 / d) if d > 256 else 1)
    most = n / 5 * 2 if d > 256 else n / 4
    p = lpq.search_plan_info(d, 8, False, n, nq, k)
    assert p[0] == 3 and p[10] * p[11] >= 3 * k * n / min(max(rows, k * n / 1500), most)
