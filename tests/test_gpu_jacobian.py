"""Rows of tdo_log_rho_jacobian against tdo_log_rho_vjp of the same configuration alone.

Both run the same layer kernels on one configuration; only the order of a few FP32
additions of per-block gradients and of the FP64 sums can differ, so a row may be off by a
few FP32 rounding steps of its terms: 1e-6 of the row's norm."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,B,budget_mib", [
    ((16, 2, 1, 64), 3, 515, 0),      # one more chunk than a full one, padded width
    ((32, 4, 1, 512), 17, 5, 24),     # chunks cut by the workspace budget
    ((64, 4, 2, 96), 32, 3, 0),       # width 64 without register feed-forward kernel
    ((64, 8, 2, 256), 31, 3, 0),
    ((64, 4, 1, 128), 33, 3, 0),      # a pass over two blocks
    ((64, 8, 1, 256), 64, 2, 0),
])
def test_jacobian_rows_equal_single_vjps(gpu, net, n, B, budget_mib, prec):
    arch = synth.arch(*net)
    params = cuda(synth.params(arch, 90 + n, "mid"))
    cfg = cuda(synth.configs(n, B, 91 + n) if n < 64 else np.random.default_rng(5).integers(0, 1 << 63, size=(B, 2), dtype=np.uint64))
    ctx = gpu.Ctx(0, budget_mib << 20)
    jac = ctx.jacobian(arch, params, n, cfg, prec)
    one = gpu.Ctx(0)
    for b in sorted({0, 1, B // 2, B - 1}):
        for part in (0, 1):
            seed = torch.zeros((1, 2), device="cuda")
            seed[0, part] = 1.0
            row = one.log_rho_vjp(arch, params, n, cfg[b:b + 1], seed, prec)
            scale = float(jac[b].norm())
            assert float((jac[b, part] - row).norm()) <= 1e-6 * scale, (b, part)
