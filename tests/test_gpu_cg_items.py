"""The split of a solve's rows into the CG loop's work items: points that do not fill the item queues evenly, items
that are no whole number of rounds over the resident blocks (so that blocks steal at the end of an iteration), one
item per few rows on teams of one, four and eight waves, and a workspace that only holds fewer chunks than the plan
would take.  Against the FP64 oracle at the precision modes' tolerances (1e-10, 1e-5), the CG on every level.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402
from paper_2510_02635_amd import workloads  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

AC = dict(f_kind=F.F_ALLEN_CAHN, fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC, gp=(0.4, 0, 0, 0), T=0.3)


@pytest.mark.parametrize("d,M,P,prec,less", [(130, 400, 37, F.F64, 0), (300, 900, 33, F.F32C, 0), (700, 800, 96, F.F32C, 0),
                                             (1030, 300, 5, F.F64, 0), (5000, 600, 3, F.F32C, 0),
                                             (5000, 600, 3, F.F32C, 20), (8200, 300, 2, F.F32C, 0)])
def test_cg_items(d, M, P, prec, less):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tol = 1e-10 if prec == F.F64 else 1e-5
    hp, op = problems(d=d, M=M, N=2, prec=prec, seed=M, solver=F.SOLVER_CG, cg_rtol=1e-12 if prec == F.F64 else 1e-7, **AC)
    x0 = workloads.points("normal_over_sqrt_d", P, d, seed=d) * 0.3
    print(f"[cg items] d={d} M={M} P={P} prec={prec} less={less}", flush=True)
    size = F.workspace_size(hp, P) - less * P * d * 8   # room for `less` partial vectors fewer per point
    u, g, st = F.solve(hp, torch.tensor(x0, device="cuda"), ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    u, g = u.cpu().numpy(), g.cpu().numpy()
    assert not st.cpu().numpy().any()
    for p in sorted({0, P // 2, P - 1}):
        ref = OS.solve_point(op, x0[p], p)
        assert abs(u[p] - ref["u"]) <= tol * abs(ref["u"]) and rel_err(g[p], ref["grad"]) <= tol
