"""Narrow kernels with a small ridge: a few particles carry the weight, the weighted design has fewer directions than
coordinates, and only the ridge keeps the level's d x d matrix positive.  Below the direct primal solve's smallest
ridge the level is the CG's, bit for bit, with no point flagged as non-finite; at it the direct solve runs and agrees
with a long double solution to the bound of a backward stable solve, 4 d eps times the condition number.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402

from _convert import problems  # noqa: E402

HJB = dict(f_kind=F.F_HJB, fp=(0.0, 0, 0, 0), g_kind=F.G_HJB_LOG, gp=(1.0, 0, 0, 0), T=0.3, N=1, seed=5)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("d,M,eps_h", [(5, 20, 0.05), (20, 40, 0.1), (64, 130, 0.05), (128, 640, 0.05)])
@pytest.mark.parametrize("ridge", [1e-9, 1e-16, 1e-20])
def test_below_the_smallest_ridge(d, M, eps_h, ridge):
    hp, _ = problems(d=d, M=M, eps_h=eps_h, ridge_rel=ridge, **HJB)
    hc, _ = problems(d=d, M=M, eps_h=eps_h, ridge_rel=ridge, solver=F.SOLVER_CG, **HJB)
    x = torch.tensor(0.3 * np.random.default_rng(d).normal(size=(300, d)), device="cuda")
    u, g, st = F.solve(hp, x)
    uc, gc, stc = F.solve(hc, x)
    torch.cuda.synchronize()
    assert not (st & 4).any() and torch.equal(st, stc) and torch.equal(u, uc) and torch.equal(g, gc)


@pytest.mark.parametrize("d,M,eps_h", [(20, 40, 0.1), (64, 130, 0.1), (100, 150, 0.05)])
def test_at_the_smallest_ridge(d, M, eps_h):
    hp, op = problems(d=d, M=M, eps_h=eps_h, ridge_rel=1e-8, **HJB)
    x0 = 0.3 * np.random.default_rng(d).normal(size=(300, d))
    u, g, st, it = F.solve(hp, torch.tensor(x0, device="cuda"), return_iters=True)
    torch.cuda.synchronize()
    assert it == [0] and not st.any()
    L = np.longdouble
    for p in (0, 150, 299):
        W = OS.brownian_path(op, p)[-1]
        Y = OS.g_eval(op, OS.positions(op, x0[p], W, 1))[0].astype(L)
        w = OS.kernel_weights(op, op.s * W, op.T).astype(L)
        D = L(op.s) * (W - w @ W.astype(L))
        B = np.sqrt(w)[:, None] * D
        A = B.T @ B + L(op.ridge_rel) * L(op.s) ** 2 * L(op.T) * np.eye(d, dtype=L)
        cond = np.linalg.cond(A.astype(np.float64))
        C = A.copy()
        z = B.T @ (np.sqrt(w) * (Y - w @ Y))
        for j in range(d):   # Cholesky and the two triangular solves, in long double
            C[j:, j] -= C[j:, :j] @ C[j, :j]
            C[j:, j] /= np.sqrt(C[j, j])
        for i in range(d):
            z[i] = (z[i] - C[i, :i] @ z[:i]) / C[i, i]
        for i in range(d - 1, -1, -1):
            z[i] = (z[i] - C[i + 1:, i] @ z[i + 1:]) / C[i, i]
        z = z.astype(np.float64)
        assert np.linalg.norm(g[p].cpu().numpy() - z) <= 4 * d * 2.0 ** -53 * cond * np.linalg.norm(z)
