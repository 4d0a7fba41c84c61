"""The tuner times the forward kernels that the tuned network runs at some batch: the layer kernel of a
single-layer network also on a few hundred samples (the loss evaluates more than n entries of each, and the
entry is kept for every later batch), none where one launch takes all layers at any batch."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("net,n,prec,timed", [
    ((64, 4, 1, 128), 16, "bf16", 4), ((32, 4, 1, 64), 8, "bf16", 4), ((64, 8, 1, 64), 12, "fp32", 2), ((64, 8, 2, 64), 40, "bf16", 4),
    ((64, 4, 2, 128), 16, "bf16", 0),
])
def test_timed_forward_launches(gpu, net, n, prec, timed):
    """Each shape is run twice over the samples, a launch per layer; no feed-forward shapes at these widths."""
    B = 64
    arch = synth.arch(*net)
    model = dict(kind=synth.ISING, n=n, V=2.0, g=1.0, gamma=1.0)
    ctx = gpu.Ctx(0)
    ctx.profile(True)
    ctx.autotune(arch, cuda(synth.params(arch, 871, "mid")), model, cuda(synth.configs(n, B, 872)), prec, "B")
    assert ctx.profile_read("fwd_layer")[1] == 2 * timed * net[2]
