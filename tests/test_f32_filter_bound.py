"""The error bound of the exact fp32 search's matrix-core filter: what splitting a product into bf16
halves drops, measured here on the worst mantissas, and the rounding of the sums fit into its constant;
and the search returns the direct kernel's bits on such mantissas (needs a real MI355X)."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2110_08919_amd import build as lpq_build


def _halves(v):
    """bf16 halves of fp32 values (round to nearest even), as fp32."""
    t = torch.as_tensor(v)
    hi = t.bfloat16().float()
    lo = (t - hi).bfloat16().float()
    return hi.double().numpy(), lo.double().numpy()


def _worst_split():
    """Largest |q x - (qh xh + qh xl + ql xh)| / |q x| over mantissas around every bf16 tie of [1, 2)."""
    ties = np.float32(1) + (2 * np.arange(128, dtype=np.float32) + 1) * np.float32(2.0 ** -8)
    v = (ties.view(np.int32)[:, None] + np.arange(-300, 301, dtype=np.int32)).reshape(-1).view(np.float32)
    v = np.concatenate([v, np.float32([1.00391388])])
    hi, lo = _halves(v)
    x = v.astype(np.float64)
    kept = hi * hi + 2 * hi * lo
    worst = np.argsort(np.abs(x * x - kept) / (x * x))[-400:]       # pairs of the worst of them
    kept = np.outer(hi[worst], hi[worst]) + np.outer(hi[worst], lo[worst]) + np.outer(lo[worst], hi[worst])
    full = np.outer(x[worst], x[worst])
    return float((np.abs(full - kept) / full).max())


def test_the_constant_covers_the_split_and_the_sums(tmp_path):
    src, exe = tmp_path / "c.hip", str(tmp_path / "c")
    src.write_text('#include <cstdio>\n#include "lpq_internal.h"\n'
                   'int main() { for (int d = 1; d <= 16384; ++d) std::printf("%.17g\\n", (double)lpq::f32_filter_constant(d)); }\n')
    subprocess.run([lpq_build.HIPCC, *lpq_build.FLAGS, str(src), "-o", exe], check=True)
    c = np.array([float(t) for t in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()])
    split, d = _worst_split(), np.arange(1, 16_385)
    assert 0.99 * 2.0 ** -15 < split < 2.0 ** -15
    # in units of (|q|^2 + |x|^2) / 2: 3 d additions of bf16 products; the norms; the directly summed distance;
    # four operations on values up to twice the unit
    rounding = 3 * d * 2.0 ** -23 * (1 + 2.0 ** -7) + d * 2.0 ** -24 + (d / 2 + 32) * 2.0 ** -24 + 8 * 2.0 ** -23
    assert np.all(c >= split + rounding)


@pytest.mark.gpu
@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("d", [1, 4, 8, 12, 33])
def test_search_of_mantissas_just_below_a_tie(metric, d):
    """Equal signs, scores a few ulps apart, half of the values exact in bf16 and half as far from it as
    they can be: the filter's scores are off in one direction only."""
    from paper_2110_08919_amd import lpq
    from test_gpu_f32_filter import _direct, _same_bits
    g = np.random.default_rng(d)
    n, nq, k = 9000, 130, 10
    near = np.float32(1.00391388).view(np.int32)
    x = (near - g.integers(0, 40, size=(n, d)).astype(np.int32)).view(np.float32)
    x[::2] = np.float32(1.0) + g.integers(0, 2, size=(n // 2, d)).astype(np.float32) * np.float32(2.0 ** -7)
    q = (near - g.integers(0, 40, size=(nq, d)).astype(np.int32)).view(np.float32)
    x, q = torch.as_tensor(x).cuda(), torch.as_tensor(q).cuda()
    _same_bits(lpq.search_f32(x, q, k, metric), _direct(lpq, x, q, k, metric))
