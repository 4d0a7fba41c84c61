"""VJP parity at the edges of the backward kernels' splits: feed-forward widths of one chunk of
32 hidden units up to the most a width takes, odd numbers of chunks, ragged last tiles, and every
head width, with the criteria of the gradient parity tests."""
import numpy as np
import pytest

from oracle import ansatz as oa
from oracle import vmc
from paper_2502_20723_amd import synth
from tests.bf16_emulation import log_rho_vjp_emulated
from tests.test_gpu_backward import assert_grad, cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,B", [
    ((16, 2, 1, 32), 4, 9), ((16, 2, 2, 96), 3, 11), ((32, 4, 1, 64), 7, 33), ((32, 4, 1, 160), 16, 5),
    ((32, 4, 1, 256), 31, 3), ((32, 4, 1, 288), 32, 3), ((32, 4, 1, 512), 33, 2), ((32, 4, 2, 128), 10, 25),
    ((64, 8, 1, 32), 5, 7), ((64, 4, 1, 96), 17, 3), ((64, 8, 1, 160), 32, 3), ((64, 4, 1, 224), 9, 4),
    ((64, 4, 2, 256), 64, 1),
])
def test_vjp_widths(gpu, net, n, B, prec):
    arch = synth.arch(*net)
    params = synth.params(arch, 400 + n, "mid")
    rng = np.random.default_rng(401 + n)
    cfg = synth.configs(n, B, 402 + n) if n < 64 else rng.integers(0, 1 << 63, size=(B, 2), dtype=np.uint64)
    seed = rng.standard_normal((B, 2)).astype(np.float32)
    got = gpu.Ctx(0).log_rho_vjp(arch, cuda(params), n, cuda(cfg), cuda(seed), prec).cpu().numpy()
    A = oa.Arch(**arch)
    ref = np.asarray(vmc.log_rho_vjp(params.astype(np.float64), A, cfg, n, seed.astype(np.float64)))
    assert_grad(prec, got, params, arch, None, cfg, None, "B", ref,
                emulate=lambda: log_rho_vjp_emulated(params, A, cfg, n, seed.astype(np.float64), prec))
