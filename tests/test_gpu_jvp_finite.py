"""What is not finite in one configuration stays out of the configurations that share its 32-row block.

An infinite tangent of a hidden unit reaches exactly the configurations with a row in which the unit is
active: a configuration whose derivative along the unit is 0 keeps 0, and the others are not finite."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("net,n,B", [((16, 2, 2, 64), 3, 23), ((32, 4, 2, 128), 8, 9), ((64, 4, 2, 96), 13, 4), ((64, 8, 3, 64), 16, 5),
                                     ((64, 8, 2, 64), 31, 4), ((64, 8, 2, 64), 40, 3)])
def test_infinite_tangent_stays_in_its_configuration(gpu, net, n, B):
    d, _, _, m = net
    arch = synth.arch(*net)
    params = synth.params(arch, 850 + n, "mid")
    b1 = 6 * d + 2 * d * d + 4 * d * d + d * m  # hidden biases of the first layer
    p, cfg = torch.from_numpy(params).cuda(), torch.from_numpy(synth.configs(n, B, 851 + n)).cuda()
    ctx = gpu.Ctx(0)
    tangent = torch.zeros(params.size, dtype=torch.float64, device="cuda")
    seen = 0
    for unit in range(b1, b1 + 8):
        for bias in np.linspace(1.0, -8.0, 91):  # until some configurations reach a positive value and some do not
            p[unit] = float(bias)
            tangent[unit] = 1.0
            active = (ctx.log_rho_jvp(arch, p, n, cfg, tangent) != 0).any(1)
            if bool(active.any()) and not bool(active.all()):
                tangent[unit] = float("inf")
                got = ctx.log_rho_jvp(arch, p, n, cfg, tangent)
                assert bool((got[~active] == 0).all()), (unit, bias)
                assert not bool(torch.isfinite(got[active]).all(1).any()), (unit, bias)
                seen += 1
        p[unit], tangent[unit] = float(params[unit]), 0.0
    assert seen > 0
