"""Encoding batches of long rows, one workgroup per row: codes, norms and padding against the CPU oracle.
Needs a real MI355X."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# rows that end inside a group of four columns, that take one and several turns of a workgroup, and more
# rows than the kernel takes (the general one is compared to the same oracle)
@pytest.mark.parametrize("n,d,bits,ld_codes", [(1, 257, 8, None), (70, 300, 4, 384), (9, 1024, 8, 1027), (5, 1027, 8, None),
                                               (33, 2048, 2, 2048), (3, 5000, 8, 5120), (16_385, 260, 8, None)])
def test_encode_long_rows(oracle, n, d, bits, ld_codes):
    from paper_2110_08919_amd import lpq
    r = np.random.default_rng(d)
    x = (r.normal(size=(n, d)) * r.uniform(0.01, 5, size=d)).astype(np.float32)
    x[0, 0], x[n - 1, d - 1], x[n // 2, d // 2] = np.nan, np.inf, -np.inf
    k, s = r.normal(size=d).astype(np.float32), r.uniform(0.5, 4, size=d).astype(np.float32)
    s[d // 3] = 0.0                     # an empty range
    gq = lpq.Quantizer(d, bits).set_params(k, k - s, k + s)
    codes, norms = gq.encode(torch.as_tensor(x).cuda(), with_norms=True, ld_codes=ld_codes)
    oq = oracle.Quantizer(d, bits).set_params(k, k - s, k + s)
    ocodes, onorms = oq.encode(x, with_norms=True)
    assert np.array_equal(codes.cpu().numpy(), ocodes) and np.array_equal(norms.cpu().numpy(), onorms)


# the last call that takes a workgroup per row and the first that does not
@pytest.mark.parametrize("n,d", [(12_098, 260), (12_099, 260), (4096, 1024), (4097, 1024)])
def test_encode_on_both_sides_of_the_rule(oracle, n, d):
    test_encode_long_rows(oracle, n, d, 8, None)
