"""The dense SR solve over the edges of its kernels (512 rows of J at a time in the column pass, rows mod
4, 128 slices of a dot product, 8 segments of a row, columns mod 256), against the same conjugate
gradients in numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("B,P", [(1, 1), (2, 7), (3, 70001), (255, 300), (256, 257), (257, 513), (515, 255), (100, 2049)])
def test_sr_solve_shapes(gpu, B, P, weighted):
    rng = np.random.default_rng(B + P)
    J, g = rng.standard_normal((B, 2, P)) + 0.5, rng.standard_normal(P)
    w = rng.uniform(0.5, 2.0, B) if weighted else np.ones(B)
    wn = (w / w.sum())[:, None, None]
    C = (np.sqrt(wn) * (J - (wn * J).sum(0))).reshape(2 * B, P)
    lam, iters = 1.0 + P / B, 5
    x, r, p = np.zeros(P), g.copy(), g.copy()
    for _ in range(iters):
        Ap = C.T @ (C @ p) + lam * p
        rs, pAp = r @ r, p @ Ap
        alpha = rs / pAp if pAp else 0.0
        x, r = x + alpha * p, r - alpha * Ap
        p = r + (r @ r / rs if rs else 0.0) * p
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    Jt = dev(J)
    got, info = gpu.Ctx(0).sr_solve(Jt, dev(g), lam, iters, dev(w) if weighted else None)
    # 64-bit sums of at most 1e5 terms in another order, five well-conditioned steps: far below 1e-10
    assert np.abs(Jt.cpu().numpy().reshape(2 * B, P) - C).max() < 1e-12
    assert np.linalg.norm(got.cpu().numpy() - x) <= 1e-10 * np.linalg.norm(x)
    assert abs(float(info[1]) - np.linalg.norm(g)) <= 1e-12 * np.linalg.norm(g)
    assert abs(float(info[0]) * np.linalg.norm(g) - np.linalg.norm(r)) <= 1e-10 * np.linalg.norm(g)
