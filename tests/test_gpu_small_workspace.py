"""Workspaces below the plan's own size: calls keep the sizes that earlier kernels asked for.

* The direct dual solve, whose M x M matrices are laid out without padding and over the CG's buffers: within the fixed
  array of the allocation-free entry point, and in P M (M + 1) doubles beyond a workspace without any CG buffer to lie
  over (cg_maxit = 1, one chunk a point).
* Its results there against the FP64 oracle (1e-10), with no CG iteration.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402
from paper_2510_02635_amd import workloads  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

AC = dict(f_kind=F.F_ALLEN_CAHN, fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC, gp=(0.4, 0, 0, 0), T=0.3)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _bytes(n, device="cuda"):
    return torch.empty(n, dtype=torch.uint8, device=device)


def _check(u, g, st, op, x0, points, tol=1e-10):
    torch.cuda.synchronize()
    u, g = u.cpu().numpy(), g.cpu().numpy()
    assert not st.any()
    for p in points:
        ref = OS.solve_point(op, x0[p], p)
        assert abs(u[p] - ref["u"]) <= tol * abs(ref["u"]) and rel_err(g[p], ref["grad"]) <= tol


@pytest.mark.parametrize("d,M,P", [(30, 17, 4000), (64, 17, 3000), (16, 17, 6000)])
def test_dual_solve_in_the_fixed_array(d, M, P):
    hp, op = problems(d=d, M=M, N=2, seed=1, **AC)
    x0 = workloads.points("normal_over_sqrt_d", P, d, seed=2)
    u = torch.empty(P, dtype=torch.float64, device="cuda")
    g = torch.empty((P, d), dtype=torch.float64, device="cuda")
    st = torch.empty(P, dtype=torch.int32, device="cuda")
    print(f"[small ws] noalloc d={d} M={M} P={P}", flush=True)
    F.solve_noalloc(hp, torch.tensor(x0, device="cuda"), u, g, st)
    _check(u, g, st, op, x0, (0, P - 1))


@pytest.mark.parametrize("d,M", [(4, 5), (15, 15), (20, 17), (40, 33), (49, 50), (60, 50), (127, 128), (130, 112)])
def test_dual_solve_in_its_square(d, M):
    P = 5
    hp, op = problems(d=d, M=M, N=2, seed=1, cg_maxit=1, **AC)
    hc, _ = problems(d=d, M=M, N=2, seed=1, cg_maxit=1, solver=F.SOLVER_CG, **AC)
    x0 = workloads.points("normal_over_sqrt_d", P, d, seed=2)
    size = F.workspace_size(hc, P) + P * M * (M + 1) * 8 + 512
    print(f"[small ws] dual d={d} M={M}", flush=True)
    u, g, st, it = F.solve(hp, torch.tensor(x0, device="cuda"), ws=_bytes(size), return_iters=True)
    assert it == [0, 0]
    _check(u, g, st, op, x0, (0, P - 1))
