"""First scan of the exact fp32 search with queries in registers (65 to 128 features, more than 256 queries): both limits of
either, rows left over behind the last 64 and 256, rows that are set aside and rows that are lost to it, strides and
alignments.  Bit for bit what the direct kernel returns.  Needs a real MI355X."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(n, d, nq, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")


def _check(x, q, k, metric):
    import f32_plan
    from paper_2110_08919_amd import lpq
    from test_gpu_f32_filter import _direct, _same_bits
    p = f32_plan.plan(x.shape[0], q.shape[0], x.shape[1], k)
    assert p["half"] and p["wq_half"] == 8 and p["nq_pad"] % 512 == 0
    _same_bits(lpq.search_f32(x, q, k, metric), _direct(lpq, x, q, k, metric))


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [
    (66_000, 128, 512, 10), (131_073, 65, 257, 1), (80_063, 127, 400, 100), (90_111, 97, 1024, 10), (70_001, 66, 1000, 33),
    (123_457, 126, 300, 7),
])
def test_sizes(metric, n, d, nq, k):
    _check(*_case(n, d, nq, n), k, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
def test_strided_and_unaligned_rows(metric):
    x, q = _case(80_000, 131, 500, 3)
    _check(x[:, 1:101], q[:, 1:101], 10, metric)


@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("rows,factor", [([99_999], 3e4), (range(5, 4096, 64), 3e5), (range(0, 99_999, 40), 1e5), ([17], float("nan")),
                                         ([64, 99_990], 1e20)])
def test_rows_that_fp16_cannot_hold(metric, rows, factor):
    x, q = _case(100_000, 128, 512, 5)
    x[list(rows)] *= factor
    _check(x, q, 10, metric)


@pytest.mark.parametrize("scale", [1e-12, 1e12])
def test_scaled_values(scale):
    x, q = _case(90_000, 100, 512, 7)
    _check(x * scale, q * scale, 10, "l2sq")
