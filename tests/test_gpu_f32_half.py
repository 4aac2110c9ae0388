"""The fp32 search's first scan, in fp16: the constant of its error covers what rounding to fp16 and the sums can
drop (CPU), and the search returns the direct kernel's bits at sizes that take it, also where that scan cannot
resolve a query or a row and leaves it to the second (needs a real MI355X)."""
import subprocess

import numpy as np
import pytest
import torch

from paper_2110_08919_amd import build as lpq_build


def test_the_constant_covers_the_rounding_and_the_sums(tmp_path):
    src, exe = tmp_path / "c.hip", str(tmp_path / "c")
    src.write_text('#include <cstdio>\n#include "lpq_internal.h"\n'
                   'int main() { for (int d = 1; d <= 16384; ++d) std::printf("%.17g\\n", (double)lpq::f32_half_filter_constant(d)); }\n')
    subprocess.run([lpq_build.HIPCC, *lpq_build.FLAGS, str(src), "-o", exe], check=True)
    c = np.array([float(t) for t in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()])
    # the worst product of two rounded values, over mantissas around every fp16 tie of [1, 2)
    ties = np.float32(1) + (2 * np.arange(1024, dtype=np.float32) + 1) * np.float32(2.0 ** -11)
    v = (ties.view(np.int32)[:, None] + np.arange(-20, 21, dtype=np.int32)).reshape(-1).view(np.float32)
    f = v.astype(np.float16).astype(np.float64)
    off = np.abs(f / v.astype(np.float64) - 1)
    rounding = (1 + off.max()) ** 2 - 1
    assert 0.99 * 2.0 ** -10 < rounding < 2.0 ** -10 + 2.0 ** -21
    # in units of (|q|^2 + |x|^2) / 2: d additions; the norms; the directly summed distance; four operations on values up
    # to twice the unit; rows too small for fp16's normal range
    d = np.arange(1, 16_385)
    sums = d * 2.0 ** -23 * (1 + 2.0 ** -9) + d * 2.0 ** -24 + (d / 2 + 32) * 2.0 ** -24 + 8 * 2.0 ** -23 + np.sqrt(d) * 2.0 ** -25
    assert np.all(c >= rounding + sums)


def _rows(n, d, nq, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((n, d), generator=g, device="cuda"), torch.randn((nq, d), generator=g, device="cuda")


def _check(x, q, k, metric):
    from paper_2110_08919_amd import lpq
    from test_gpu_f32_filter import _direct, _same_bits
    _same_bits(lpq.search_f32(x, q, k, metric), _direct(lpq, x, q, k, metric))


# query tiles of 64, 128 and 256; rows of 1 to 3 features, that end inside a 16-byte load, inside a stage and at its end,
# and that are not 16-byte aligned; a corpus that ends inside a tile
@pytest.mark.gpu
@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("n,d,nq,k", [(1_000_003, 3, 64, 10), (1_000_000, 1, 60, 3), (520_000, 65, 128, 10), (260_001, 127, 129, 100),
                                      (130_000, 100, 257, 10), (65_537, 515, 130, 7), (200_000, 32, 700, 1)])
def test_first_scan_returns_the_direct_kernels_bits(metric, n, d, nq, k):
    x, q = _rows(n, d, nq, d)
    _check(x, q, k, metric)


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1e-14, 1e-6, 300.0, 1e9])
def test_queries_and_rows_of_any_scale(scale):
    """Also queries that are zero, far larger and far smaller than the others of their tile."""
    x, q = _rows(130_000, 70, 300, 1)
    x, q = x * scale, q * scale
    _check(x, q, 10, "l2sq")
    _check(x * 1000.0, q, 10, "ip")
    q[5], q[70], q[131] = 0.0, q[70] * 1e-12, q[131] * 1e4
    q[200], q[299] = 1e-19, q[299] * 1e-9
    for metric in ("l2sq", "ip"):
        _check(x, q, 10, metric)


@pytest.mark.gpu
def test_rows_and_queries_the_first_scan_leaves_to_the_second():
    x, q = _rows(130_000, 70, 300, 2)
    big = x.clone()
    big[77_777] *= 1e5                      # too large for fp16
    big[3] *= 1e3
    for metric in ("l2sq", "ip"):
        _check(big, q, 10, metric)
    far = 0.05 * x + 20.0                   # within the first scan's error of each other
    mixed = torch.where(torch.arange(130_000, device="cuda")[:, None] % 2 == 0, far, x)
    qm = torch.where(torch.arange(300, device="cuda")[:, None] % 100 == 99, 0.05 * q + 20.0, q)
    _check(mixed, qm, 10, "l2sq")
    _check(far, 0.05 * q + 20.0, 10, "l2sq")
    dup = x.clone()
    dup[20_000:60_000] = dup[0]             # more equal rows than a region holds, found by few queries
    q[7] = dup[0]
    _check(dup, q, 10, "l2sq")


# one row, as many as a wave of the scan sets aside (all of them in the rows of the same wave) and more, and rows that only
# scaled rows can hold
@pytest.mark.gpu
@pytest.mark.parametrize("metric", ["l2sq", "ip"])
@pytest.mark.parametrize("norm,long,factor,resolved", [
    (1.0, [77_777], 3e4, True), (85.0, [3, 255, 256, 129_999], 60.0, True), (85.0, [129_999], 1e4, True),
    (85.0, range(7, 16 * 256, 256), 50.0, True), (40.0, range(0, 129_999, 256), 2000.0, None),
    (85.0, range(5, 129_999, 50), 60.0, None), (1e-9, [500], 1e7, True), (1e3, [9], 1e12, False)])
def test_rows_of_large_norm_cost_only_themselves(metric, norm, long, factor, resolved):
    """A row that fp16 cannot hold is set aside: the first scan still resolves the queries of its tile."""
    import f32_plan
    from paper_2110_08919_amd import lpq
    from test_gpu_f32_filter import _direct, _same_bits
    x, q = _rows(130_000, 128, 300, 3)
    x, q = x * norm, q * norm
    x[list(long)] *= factor
    got, p, ws = f32_plan.search(x, q, 10, metric)
    _same_bits(got, _direct(lpq, x, q, 10, metric))
    again, hard = f32_plan.words(p, ws, "off_again", 300), f32_plan.words(p, ws, "off_hard", p["nq_pad"] // 128)
    assert p["half"]
    if resolved is not None:
        left = (again != 0) | (hard[torch.arange(300, device="cuda") // 128] != 0)
        assert bool(left.any()) != resolved


def _some_hard(rows):
    """1M x 128, every second row shifted by 5, and so the queries `rows` of 1000, which the first scan cannot resolve where
    they are near many of the shifted rows."""
    x, q = _rows(1_000_000, 128, 1000, 1)
    x[::2] += 5.0
    q[list(rows)] += 5.0
    return x, q


@pytest.mark.gpu
def test_a_few_hard_queries_cost_no_more_than_the_second_scan_of_all():
    """A few of 1000 queries hard, in 3 of 8 tiles: 1.36 times as long as with all of them hard when the workgroups with work met
    on half of the shader engines."""
    import f32_plan
    from paper_2110_08919_amd import lpq
    x, few = _some_hard(range(64, 1000, 128))
    _, every = _some_hard(range(1000))
    assert f32_plan.best_ms(lambda: lpq.search_f32(x, few, 10, "l2sq")) <= 1.15 * f32_plan.best_ms(lambda: lpq.search_f32(x, every, 10, "l2sq"))


@pytest.mark.gpu
@pytest.mark.parametrize("tiles,left", [((3,), 0), ((0, 7), 0), ((1, 2, 6), 616), ((0, 1, 2, 3, 4, 6), 232), (range(8), 0)])
def test_queries_beside_many_hard_tiles_are_left_to_the_second_scan(tiles, left):
    import f32_plan
    from paper_2110_08919_amd import lpq
    from test_gpu_f32_filter import _direct, _same_bits
    x, q = _some_hard([128 * t + i for t in tiles for i in range(40)])
    x = x[:260_000].contiguous()
    got, p, ws = f32_plan.search(x, q, 10, "l2sq")
    _same_bits(got, _direct(lpq, x, q, 10, "l2sq"))
    hard = f32_plan.words(p, ws, "off_hard", 8)
    assert hard.nonzero().flatten().tolist() == list(tiles)
    assert int((f32_plan.words(p, ws, "off_again", 1000) != 0).sum()) == left
