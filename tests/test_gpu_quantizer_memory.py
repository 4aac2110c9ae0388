"""Device memory a quantizer holds: its constants and the partial results of a calibration, whatever the
mode it was calibrated in.  Needs a real MI355X."""
import gc

import numpy as np
import pytest
import torch

from paper_2110_08919_amd import lpq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [None, "minmax", "quantile"])
def test_quantizers_hold_little_memory(mode):
    d, count = 128, 40
    x = torch.randn((50_000, d), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    def make():
        q = lpq.Quantizer(d, 8)
        return q.set_params(np.zeros(d), -np.ones(d), np.ones(d)) if mode is None else q.calibrate(x, mode, "per_feature", 0.001)
    first = make()
    gc.collect()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    held = [make() for _ in range(count)]
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    # partial results of 1024 workgroups (2.1 MB), histograms of the general quantile path (0.5 MB), rounded up
    assert used <= count * (4 << 20), f"{used / count / 2 ** 20:.1f} MB each"
    assert len(held) == count and first is not None
