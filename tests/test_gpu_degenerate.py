"""Clouds without spread: the geometric family at x0 = 0 stays there, so every level's system and its right-hand side
are zero.  The slope is zero and u that of the equation without diffusion, in the direct solves as in the CG; a point
off the origin in the same call keeps its values.  Against the FP64 oracle for that point and the CG for the other.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

AC = dict(f_kind=F.F_ALLEN_CAHN, fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC, gp=(0.4, 0, 0, 0), T=0.3)


@pytest.mark.parametrize("d,M", [(10, 40), (10, 8), (100, 200)])
@pytest.mark.parametrize("prec,tol", [(F.F64, 1e-10), (F.F32C, 1e-5)])
def test_geometric_family_at_the_origin(d, M, prec, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hp, op = problems(d=d, M=M, N=3, seed=1, prec=prec, **AC)
    hc, _ = problems(d=d, M=M, N=3, seed=1, prec=prec, solver=F.SOLVER_CG, **AC)
    x0 = np.zeros((2, d))
    x0[1] = 0.3 + 0.1 * np.cos(np.arange(d))
    xt = torch.tensor(x0, device="cuda")
    u, g, st = F.solve_coef(hp, xt, 0.05, 0.2)
    uc, gc, stc = F.solve_coef(hc, xt, 0.05, 0.2)
    torch.cuda.synchronize()
    assert not st.any() and not stc.any()
    assert not g[0].any() and abs(u[0] - uc[0]).item() <= tol * abs(uc[0].item())
    ref = OS.solve_point_coef(op, x0[1], 1, (0.05, 0.2, 0.0, 0.0))
    assert abs(u[1].item() - ref["u"]) <= tol * abs(ref["u"]) and rel_err(g[1].cpu().numpy(), ref["grad"]) <= tol
