"""The forward in one launch against the forward layer by layer: the same bits.  Which of the two a
call takes depends on the batch (a single layer: up to one tile per pair of waves), so a large batch
and its first configurations, or chains, take different ones.  One tile holds 32 // n configurations; 256 CUs of 4 pairs of waves each."""
import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# (network, n, large batch, parts): the parts take the other route, and end in ragged tiles
CASES = [((64, 8, 1, 256), 32, 1031, (1, 257, 515, 1024)), ((64, 4, 1, 96), 17, 1025, (3, 300)), ((32, 4, 1, 512), 8, 4101, (9, 2050)),
         ((16, 2, 1, 64), 3, 10300, (7, 2561, 5121)), ((64, 4, 1, 128), 31, 1030, (2,)), ((16, 2, 1, 32), 5, 6150, (1, 4000))]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,B,parts", CASES + [((64, 8, 2, 256), 11, 600, (5, 511)), ((64, 8, 3, 64), 32, 300, (256, 255))])
def test_log_rho_same_bits(gpu, net, n, B, parts, prec):
    arch = synth.arch(*net)
    params, cfg = cuda(synth.params(arch, 800 + n, "mid")), cuda(synth.configs(n, B, 801 + n))
    ctx = gpu.Ctx(0)
    whole = ctx.log_rho(arch, params, n, cfg, prec)
    assert bool(torch.isfinite(whole).all())
    for k in parts:
        assert torch.equal(ctx.log_rho(arch, params, n, cfg[:k].contiguous(), prec), whole[:k]), k


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("net,n,C,parts", CASES)
def test_chains_same_states(gpu, net, n, C, parts, prec):
    """Two sweeps of the first chains, alone and among more chains than the one launch takes."""
    arch = synth.arch(*net)
    params, cfg = cuda(synth.params(arch, 810 + n, "mid")), cuda(synth.configs(n, C, 811 + n))
    ctx = gpu.Ctx(0)

    def run(k):
        state = cfg[:k].clone()
        lr = ctx.log_rho(arch, params, n, state, prec)
        samples, counter = ctx.sample(arch, params, n, state, lr, 77, 5, 2, 0.4, prec)
        diag = cfg[:k, 0].clone()  # (a view for k = 1 otherwise, and the chains move in place)
        dlr = ctx.log_rho(arch, params, n, torch.stack([diag, diag], 1), prec)
        dsamples, dcounter = ctx.sample_diag(arch, params, n, diag, dlr, 78, 5, 2, prec)
        assert (counter, dcounter) == (5 + 4 * n, 5 + 2 * n)
        return [t.cpu().numpy() for t in (samples, state, lr, dsamples, diag, dlr)]

    whole = run(C)
    for k in parts:
        for i, (got, ref) in enumerate(zip(run(k), whole)):
            assert np.array_equal(got, ref[:, :k] if i in (0, 3) else ref[:k]), (k, i)


# batches in which a BF16 wave holds both tiles of a pair: 5 to 8 pairs a workgroup, one round or more, ragged ends
TWO = [((64, 8, 2, 256), 32, 1025, (1024, 1)), ((64, 8, 2, 256), 31, 3300, (511,)), ((64, 4, 2, 96), 9, 3 * 1500 + 1, (3000,)),
       ((32, 4, 3, 128), 8, 4 * 3500 - 1, (1000, 4096)), ((16, 2, 2, 32), 3, 10 * 6000 + 3, (10240,)), ((64, 4, 2, 256), 16, 4096, (1,))]


@pytest.mark.parametrize("net,n,B,parts", TWO)
def test_two_tiles_per_wave(gpu, net, n, B, parts):
    """log rho has the same bits as in a batch whose waves hold one tile."""
    arch = synth.arch(*net)
    params, cfg = cuda(synth.params(arch, 820 + n, "mid")), cuda(synth.configs(n, B, 821 + n))
    ctx = gpu.Ctx(0)
    whole = ctx.log_rho(arch, params, n, cfg, "bf16")
    assert bool(torch.isfinite(whole).all())
    for k in parts:
        assert torch.equal(ctx.log_rho(arch, params, n, cfg[:k].contiguous(), "bf16"), whole[:k]), k


@pytest.mark.parametrize("net,n,C,parts", [((64, 8, 2, 64), 32, 1029, (1024,)), ((64, 4, 2, 256), 13, 2 * 3300 - 1, (700,)),
                                           ((32, 4, 3, 96), 8, 4 * 1300 + 1, (4096, 5)), ((16, 2, 2, 64), 3, 10 * 1500, (10001,))])
def test_two_tiles_per_wave_chains(gpu, net, n, C, parts):
    test_chains_same_states(gpu, net, n, C, parts, "bf16")


@pytest.mark.parametrize("net,n,B", [((64, 8, 2, 64), 32, 16385), ((64, 4, 2, 256), 16, 2 * 17000 - 1), ((32, 4, 2, 96), 9, 3 * 16500 + 2),
                                     ((16, 2, 2, 32), 3, 10 * 20001 - 7)])
def test_two_tiles_per_wave_with_activations(gpu, net, n, B):
    """The gradient of more than 64 pairs of tiles per CU against the sum over batches whose waves hold
    one tile: the same terms, with the same bits, in another grouping.  A workgroup sums at most 32 B / 256
    rows in FP32 (the rest is FP64): 2^-24 sqrt(32 B / 256) = 1e-5 of the sum at the largest B, and 1e-4 of
    the largest component leaves room for cancellation; a misplaced tile gives O(1)."""
    arch = synth.arch(*net)
    params, cfg = cuda(synth.params(arch, 830 + n, "mid")), cuda(synth.configs(n, B, 831 + n))
    seed = cuda(np.random.default_rng(832 + n).standard_normal((B, 2)).astype(np.float32))
    ctx = gpu.Ctx(0)
    grad = ctx.log_rho_vjp(arch, params, n, cfg, seed, "bf16")
    step = 16 * 256 * (32 // n)
    parts = sum(ctx.log_rho_vjp(arch, params, n, cfg[i:i + step].contiguous(), seed[i:i + step].contiguous(), "bf16") for i in range(0, B, step))
    assert float((grad - parts).abs().max()) <= 1e-4 * float(parts.abs().max())
