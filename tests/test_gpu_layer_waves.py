"""The FP32 layer kernel with 4 and with 8 waves a workgroup: the same bits.  Which of them a batch takes
depends on its rounds of the chip (1024 tiles with 4 waves, 2048 with 8), so a large batch and its first
configurations take different ones; a spanning pass of width 64 has 4 only."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth
from tests.test_gpu_sum_order import network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("net,n,parts", [
    ((32, 4, 3, 128), 50, (3, 511, 1025, 2001, 3072)), ((16, 2, 2, 96), 33, (1, 1023, 1100, 3000)), ((32, 4, 1, 64), 64, (1600, 2048)),
    ((64, 4, 1, 256), 32, (1025, 1500, 2048, 2500, 4096)), ((64, 8, 1, 96), 17, (1100, 1900)), ((32, 4, 1, 128), 16, (2 * 1025 + 1, 2 * 2040, 2 * 2500)),
    ((16, 2, 1, 32), 5, (6 * 1200 + 1, 6 * 1800)), ((64, 4, 2, 256), 37, (5, 600, 1100)), ((64, 8, 3, 64), 60, (1, 513)),
])
def test_log_rho_of_parts(gpu, net, n, parts):
    B = parts[-1] + 7
    arch, params, cfg, _ = network(net, n, B, 960)
    ctx = gpu.Ctx(0)
    assert gpu.lib().tdo_test_layer_forward(ctx.h, 1) == 0
    whole = ctx.log_rho(arch, params, n, cfg, "fp32")
    assert bool(torch.isfinite(whole).all())
    for k in parts:
        assert torch.equal(ctx.log_rho(arch, params, n, cfg[:k].contiguous(), "fp32"), whole[:k]), k
