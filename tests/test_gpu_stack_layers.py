"""The forward in one launch against the layer kernel for networks of several layers: the same bits, in log rho, in
chains, and in the activations kept for the backward pass (through every gradient, whose kernels are the same).
A context that never takes the one launch gives the other side."""
import numpy as np
import pytest
import torch

from oracle import ansatz as oa
from paper_2502_20723_amd import synth
from tests.parity import log_rho_err

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


@pytest.fixture
def both(gpu):
    """(one launch, layer by layer)"""
    stack, layers = gpu.Ctx(0), gpu.Ctx(0)
    assert gpu.lib().tdo_test_layer_forward(layers.h, 1) == 0
    return stack, layers


def launches(ctx, call):
    ctx.profile(True)
    out = call()
    k = ctx.profile_read("fwd_layer")[1]
    ctx.profile(False)
    return out, k


# one tile per wave on a few CUs, on all, and (BF16) two tiles per wave in one round and more; ragged ends
LOG_RHO = [((64, 8, 4, 256), 32, (1, 300, 1025, 5001)), ((64, 8, 2, 64), 31, (511, 3300)), ((64, 4, 3, 96), 9, (7, 3 * 1100 + 2, 3 * 4000 + 1)),
           ((64, 4, 2, 256), 16, (2 * 1000 - 1, 4096)), ((32, 4, 3, 512), 8, (9, 4 * 1500 + 3)), ((32, 4, 4, 64), 20, (1030,)),
           ((16, 2, 4, 32), 3, (10 * 1024, 10 * 1500 + 7)), ((16, 2, 16, 64), 5, (601,))]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,batches", LOG_RHO)
def test_log_rho(gpu, both, net, n, batches, prec):
    stack, layers = both
    arch = synth.arch(*net)
    params = cuda(synth.params(arch, 900 + n, "mid"))
    for B in batches:
        cfg = cuda(synth.configs(n, B, 901 + n))
        a, one = launches(stack, lambda: stack.log_rho(arch, params, n, cfg, prec))
        b, many = launches(layers, lambda: layers.log_rho(arch, params, n, cfg, prec))
        assert many == one * net[2]
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b), B


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,C", [((64, 8, 4, 256), 32, 33), ((64, 8, 2, 64), 32, 1029), ((64, 4, 3, 96), 9, 100), ((64, 4, 2, 256), 13, 2 * 1100 - 1),
                                     ((32, 4, 4, 128), 8, 4 * 1100 + 1), ((16, 2, 3, 64), 3, 10 * 1100)])
def test_chains(gpu, both, net, n, C, prec):
    arch = synth.arch(*net)
    params, cfg = cuda(synth.params(arch, 910 + n, "mid")), cuda(synth.configs(n, C, 911 + n))
    out = []
    for ctx in both:
        state = cfg.clone()
        lr = ctx.log_rho(arch, params, n, state, prec)
        samples, _ = ctx.sample(arch, params, n, state, lr, 91, 3, 2, 0.4, prec)
        diag = cfg[:, 0].clone()
        dlr = ctx.log_rho(arch, params, n, torch.stack([diag, diag], 1), prec)
        dsamples, _ = ctx.sample_diag(arch, params, n, diag, dlr, 92, 3, 2, prec)
        out.append([t.cpu().numpy() for t in (samples, state, lr, dsamples, diag, dlr)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


# the last batch of each BF16 case has more than 64 pairs of tiles per CU: two tiles per wave
GRAD = [((64, 8, 2, 64), 32, (3, 1025, 16385)), ((64, 4, 3, 256), 16, (2 * 700 - 1, 2 * 16500 + 1)), ((32, 4, 2, 96), 9, (31, 3 * 16400 + 2)),
        ((16, 2, 4, 32), 3, (10 * 300 + 1, 10 * 16400 + 3))]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,batches", GRAD)
def test_reverse_mode(gpu, both, net, n, batches, prec):
    stack, layers = both
    arch = synth.arch(*net)
    params = cuda(synth.params(arch, 920 + n, "mid"))
    for B in batches if prec == "bf16" else batches[:-1]:
        cfg = cuda(synth.configs(n, B, 921 + n))
        cot = cuda(np.random.default_rng(922 + n).standard_normal((B, 2)).astype(np.float32))
        a = stack.log_rho_vjp(arch, params, n, cfg, cot, prec)
        assert torch.equal(a, layers.log_rho_vjp(arch, params, n, cfg, cot, prec)), B


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,B", [((64, 8, 4, 256), 32, 40), ((64, 4, 2, 256), 11, 300), ((32, 4, 2, 128), 8, 500), ((16, 2, 2, 64), 4, 256)])
def test_loss_and_jacobian(gpu, both, net, n, B, prec):
    """The entries' number on the device, log rho beside the activations, one configuration a block."""
    arch = synth.arch(*net)
    params, cfg = cuda(synth.params(arch, 930 + n, "mid")), cuda(synth.configs(n, B, 931 + n))
    model = dict(kind=synth.XYZ, n=n, Jx=0.9, Jy=1.0, Jz=1.1, gamma=1.0)
    a, b = ([*ctx.loss_grad(arch, params, model, cfg, None, prec), ctx.jacobian(arch, params, n, cfg[:33], prec)] for ctx in both)
    for x, y in zip(a, b):
        assert x is None and y is None or torch.equal(x, y)


@pytest.mark.parametrize("n,B", [(32, 70), (12, 333)])
def test_layer_kernel_behind_the_first_layer(gpu, n, B):
    """A BF16 feed-forward width whose weights one launch cannot hold, against the oracle at the stated bound."""
    arch = synth.arch(64, 8, 2, 288)
    params, cfg = synth.params(arch, 940 + n, "mid"), synth.configs(n, B, 941 + n)
    got = gpu.Ctx(0).log_rho(arch, cuda(params), n, cuda(cfg), "bf16").cpu().numpy()
    assert log_rho_err(got, oa.log_rho(params.astype(np.float64), oa.Arch(**arch), cfg, n).numpy()) < 2e-2
