"""The order of the sums behind the SR updates.

A conjugate-gradient solve that stops after a few iterations of an ill-conditioned system carries a
changed rounding of its operator or of its own sums into the update, by orders of magnitude more than
the rounding itself (J changed by 2e-16: up to 1e-5 of the update).  The order of these sums is
therefore part of what the calls return.  The digests below are of the outputs in that order, on inputs
made from seeds, bit for bit: of the forward-mode pass with the FP32 sums that k_jvp_layer states, of the
FP64 sums of the solve, and of the attention's reverse mode over two blocks."""
import hashlib

import numpy as np
import pytest
import torch

from paper_2502_20723_amd import synth

pytestmark = pytest.mark.gpu


def cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def digest(outputs):
    return hashlib.sha256(b"".join(t.cpu().numpy().tobytes() for t in outputs)).hexdigest()[:16]


def network(net, n, B, seed):
    arch = synth.arch(*net)
    rng = np.random.default_rng([seed, n])
    cfg = rng.integers(0, 1 << 63, size=(B, 2), dtype=np.uint64) * np.uint64(2) + rng.integers(0, 2, size=(B, 2), dtype=np.uint64)
    cfg = cfg & np.uint64((1 << n) - 1)
    params = synth.params(arch, seed + n, "mid")
    return arch, cuda(params), cuda(cfg), cuda(rng.standard_normal(params.size))


def jvp(tdo, net, n, B):
    arch, params, cfg, tangent = network(net, n, B, 4000)
    return [tdo.Ctx(0).log_rho_jvp(arch, params, n, cfg, tangent)]


def solve(tdo, B, P, iters, weighted):
    """A stopped solve with a small shift: the rows of J lie near a few directions."""
    rng = np.random.default_rng([4200, B, P])
    J = rng.standard_normal((B, 2, P)) * 0.01 + rng.standard_normal((B, 2, 1)) * rng.standard_normal(P)
    grad, w = cuda(rng.standard_normal(P)), cuda(rng.uniform(0.5, 2.0, B)) if weighted else None
    jac = cuda(J)
    return [*tdo.Ctx(0).sr_solve(jac, grad, 1e-3, iters, w), jac]


def conv_rows(tdo, net, n, B, prec):
    """The log-derivatives of the convolutions, which lie behind every layer's reverse mode."""
    arch, params, cfg, _ = network(net, n, B, 4400)
    return [tdo.Ctx(0).jacobian(arch, params, n, cfg, prec)[..., :6 * net[0] + 2 * net[0] ** 2].contiguous()]


JVP = [((16, 2, 1, 64), 3, 61), ((16, 1, 2, 32), 9, 7), ((16, 2, 3, 64), 33, 5), ((32, 4, 2, 128), 8, 37), ((32, 2, 1, 96), 20, 3),
       ((32, 4, 4, 64), 64, 9), ((64, 4, 2, 256), 16, 33), ((64, 4, 1, 512), 37, 5), ((64, 8, 3, 128), 5, 40), ((64, 8, 4, 256), 32, 17),
       ((64, 8, 2, 256), 50, 6)]


# rows 2 mod 4 and 0 mod 4, below and above one load of the column pass, P below and above the slices
SOLVE = [(1, 1, 3, False), (2, 300, 9, True), (7, 1001, 23, False), (24, 5003, 15, True), (256, 700, 12, False), (257, 2050, 30, False),
         (600, 257, 6, True), (40, 70001, 20, False)]


# passes over two blocks in the kernels of widths 16 and 32 and of FP32: dK and dV of both query blocks in one sum
SPAN = [((16, 2, 2, 64), 64, 9, "bf16"), ((32, 4, 4, 64), 64, 25, "bf16"), ((32, 4, 2, 128), 50, 9, "bf16"), ((32, 4, 3, 128), 63, 5, "fp32"),
        ((64, 8, 3, 128), 64, 5, "fp32"), ((64, 8, 2, 256), 37, 4, "fp32")]


def cases():
    c = {"jvp %s n=%d" % ("-".join(map(str, a[0])), a[1]): (jvp, a) for a in JVP}
    c.update({"solve B=%d P=%d" % a[:2]: (solve, a) for a in SOLVE})
    c.update({"rows %s n=%d %s" % ("-".join(map(str, a[0])), a[1], a[3]): (conv_rows, a) for a in SPAN})
    return c


WANT = {
    "jvp 16-2-1-64 n=3": "3f0e5cdeaf286006",
    "jvp 16-1-2-32 n=9": "3f629f8cc3db478f",
    "jvp 16-2-3-64 n=33": "e1727b1260e2c274",
    "jvp 32-4-2-128 n=8": "aef33a108e2aa2cf",
    "jvp 32-2-1-96 n=20": "95d265a1eda4ba85",
    "jvp 32-4-4-64 n=64": "3ff97b4020a18ebe",
    "jvp 64-4-2-256 n=16": "e2b94a1d4248f0bd",
    "jvp 64-4-1-512 n=37": "bb49e60b29d20d09",
    "jvp 64-8-3-128 n=5": "10a47c40f317cb7c",
    "jvp 64-8-4-256 n=32": "f2d992d54d11c186",
    "jvp 64-8-2-256 n=50": "f3ca638918254641",
    "solve B=1 P=1": "157dee46fa47f596",
    "solve B=2 P=300": "d1b20d28d1b944ee",
    "solve B=7 P=1001": "1374bd8bf4960244",
    "solve B=24 P=5003": "a23a8c2b31944b66",
    "solve B=256 P=700": "f128f9990e35fc65",
    "solve B=257 P=2050": "387b6cbb3af267ad",
    "solve B=600 P=257": "2c6476c9aee2cba4",
    "solve B=40 P=70001": "36eb263fb000fd35",
    "rows 16-2-2-64 n=64 bf16": "f41d207db3deb4c3",
    "rows 32-4-4-64 n=64 bf16": "bb225ae0d6e1648d",
    "rows 32-4-2-128 n=50 bf16": "ddbc0646eb41623c",
    "rows 32-4-3-128 n=63 fp32": "3dde12f5f24929d9",
    "rows 64-8-3-128 n=64 fp32": "224614048830d188",
    "rows 64-8-2-256 n=37 fp32": "91a1754e35360ecf",
}


@pytest.mark.parametrize("name", list(cases()))
def test_bits(gpu, name):
    f, args = cases()[name]
    assert digest(f(gpu, *args)) == WANT[name]


@pytest.mark.parametrize("net,n,B,prec", [
    ((16, 2, 1, 64), 3, 13, "fp32"), ((16, 2, 3, 32), 17, 3, "bf16"), ((32, 4, 2, 128), 8, 5, "fp32"), ((32, 4, 1, 512), 32, 3, "bf16"),
    ((64, 4, 2, 256), 16, 4, "fp32"), ((64, 8, 1, 96), 31, 2, "fp32"), ((64, 8, 2, 256), 32, 3, "bf16"), ((64, 4, 1, 256), 47, 2, "bf16"),
])
def test_jacobian_rows_are_single_vjps(gpu, net, n, B, prec):
    """Bit for bit.  (A pass over two blocks in the kernels of widths 16 and 32 and of FP32 is left out: a workgroup
    takes all four blocks of a row there and two of a single reverse-mode pass.)"""
    arch, params, cfg, _ = network(net, n, B, 4300)
    jac = gpu.Ctx(0).jacobian(arch, params, n, cfg, prec)
    ctx = gpu.Ctx(0)
    for b in range(B):
        for part in (0, 1):
            seed = torch.zeros((1, 2), device="cuda")
            seed[0, part] = 1.0
            assert torch.equal(jac[b, part], ctx.log_rho_vjp(arch, params, n, cfg[b:b + 1], seed, prec)), (b, part)
