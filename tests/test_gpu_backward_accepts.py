"""Which feed-forward widths the backward takes: every multiple of 32 up to 512 at widths 16 and 32, up to
256 at width 64 (its chunks of 32 hidden units are held in registers, one for each of 8 waves).  What it does
not take is refused by every call that needs it before a kernel is launched."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("d,heads", [(16, 2), (32, 4), (64, 4), (64, 8)])
def test_feed_forward_widths(gpu, d, heads, prec):
    n, B = 5, 2
    cfg = torch.from_numpy(synth.configs(n, B, 881)).cuda()
    cot = torch.ones((B, 2), device="cuda")
    model = dict(kind=synth.ISING, n=n, V=2.0, g=1.0, gamma=1.0)
    ctx = gpu.Ctx(0)
    for mlp in range(32, 513, 32):
        arch = synth.arch(d, heads, 1, mlp)
        params = torch.from_numpy(synth.params(arch, 880, "mid")).cuda()
        calls = (lambda: ctx.log_rho_vjp(arch, params, n, cfg, cot, prec), lambda: ctx.jacobian(arch, params, n, cfg, prec),
                 lambda: ctx.loss_grad(arch, params, model, cfg, None, prec)[1])
        for call in calls:
            if d < 64 or mlp <= 256:
                assert bool(torch.isfinite(call()).all()), mlp
            else:
                ctx.profile(True)
                with pytest.raises(gpu.TdoError, match="mlp %d" % mlp):
                    call()
                assert ctx.profile_read("fwd_layer")[1] == 0
                ctx.profile(False)
