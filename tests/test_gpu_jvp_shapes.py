"""tdo_log_rho_jvp at the edges of its kernel: padded widths and heads, head widths 8 and 16 at each
width, several configurations a block, a pass over two blocks with a ragged last workgroup, and
chunks and weight packing cut by the workspace.  The reference is the oracle's Jacobian times the
tangent; an FP32 evaluation is a few hundred rounding steps of its summands off, and 1e-3 is the
stated gradient bound."""
import numpy as np
import pytest
import torch

from oracle import ansatz as oa
from oracle import sr as osr
from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def inputs(net, n, B):
    arch = synth.arch(*net)
    rng = np.random.default_rng(700 + n)
    cfg = synth.configs(n, B, 701 + n) if n < 64 else rng.integers(0, 1 << 63, size=(B, 2), dtype=np.uint64)
    params = synth.params(arch, 702 + n, "mid")
    return arch, params, cfg, rng.standard_normal(params.size) * 0.1


@pytest.mark.parametrize("net,n,B", [
    ((16, 1, 1, 32), 3, 23), ((16, 2, 2, 64), 31, 2), ((32, 2, 1, 96), 10, 7), ((32, 2, 1, 64), 33, 3),
    ((32, 4, 2, 128), 32, 3), ((64, 4, 1, 512), 5, 13), ((64, 8, 1, 32), 64, 3), ((64, 4, 2, 256), 47, 1),
])
def test_jvp_shapes(gpu, net, n, B):
    arch, params, cfg, tan = inputs(net, n, B)
    J = osr.jacobian(params.astype(np.float64), oa.Arch(**arch), cfg, n)
    ref = np.stack([J[:, 0] @ tan, J[:, 1] @ tan], axis=1)
    got = gpu.Ctx(0).log_rho_jvp(arch, cuda(params), n, cuda(cfg), cuda(tan)).cpu().numpy()
    assert np.linalg.norm(got - ref) < 1e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [8, 40])
def test_jvp_small_workspace_is_bit_identical(gpu, n):
    """One layer's weights at a time and chunks of a few configurations give the same values."""
    arch, params, cfg, tan = inputs((64, 4, 3, 256), n, 61)
    args = (arch, cuda(params), n, cuda(cfg), cuda(tan))
    assert torch.equal(gpu.Ctx(0, 1 << 20).log_rho_jvp(*args), gpu.Ctx(0).log_rho_jvp(*args))
