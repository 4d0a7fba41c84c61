"""The same call twice gives the same bits: the gradients of the FP32 kernels and of the BF16 ones at widths 16 and
32 are sums in a fixed order, also over many workgroups, chunks and spanning passes."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("net,n,B,prec", [
    ((16, 2, 2, 64), 4, 3001, "fp32"), ((16, 2, 2, 64), 36, 200, "bf16"), ((32, 4, 2, 128), 8, 4096, "bf16"), ((32, 4, 2, 512), 33, 150, "fp32"),
    ((32, 4, 3, 96), 21, 777, "bf16"), ((64, 4, 2, 256), 16, 1500, "fp32"), ((64, 4, 2, 256), 37, 300, "fp32"), ((64, 8, 1, 96), 64, 200, "fp32"),
    ((64, 8, 2, 96), 32, 700, "bf16"),
])
def test_gradients_repeat(gpu, net, n, B, prec):
    arch = synth.arch(*net)
    params = cuda(synth.params(arch, 950 + n, "mid"))
    cfg = cuda(synth.configs(n, B, 951 + n) if n < 64 else np.random.default_rng(5).integers(0, 1 << 63, size=(B, 2), dtype=np.uint64))
    cot = cuda(np.random.default_rng(952 + n).standard_normal((B, 2)).astype(np.float32))
    model = dict(kind=synth.ISING, n=n, V=2.0, g=1.1, gamma=1.0)
    few = cfg[:max(8, 2000 // n)].contiguous()

    def outputs(ctx):
        loss, grad, _ = ctx.loss_grad(arch, params, model, few, None, prec)
        return [ctx.log_rho_vjp(arch, params, n, cfg, cot, prec), loss, grad, ctx.jacobian(arch, params, n, cfg[:7].contiguous(), prec)]

    ctx = gpu.Ctx(0)
    first = outputs(ctx)
    for again in (outputs(ctx), outputs(gpu.Ctx(0))):
        for a, b in zip(first, again):
            assert torch.equal(a, b)
