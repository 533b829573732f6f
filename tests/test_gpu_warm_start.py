"""The CG's start from the two levels before (M >= 2 d) against the start from one (M < 2 d), around the border, over
enough levels to use both slopes, with and without the tape and under a fixed iteration count.  Against the FP64
oracle at the precision modes' tolerances (1e-10, 1e-5).
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402
from paper_2510_02635_amd import workloads  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

AC = dict(f_kind=F.F_ALLEN_CAHN, fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC, gp=(0.4, 0, 0, 0), T=0.3)
HJB = dict(f_kind=F.F_HJB, fp=(0.8, 0, 0, 0), g_kind=F.G_HJB_LOG, gp=(1.0, 0, 0, 0), T=0.4)


@pytest.mark.parametrize("d,M,N,fam", [(60, 119, 5, AC), (60, 120, 5, HJB), (60, 121, 2, AC), (150, 600, 7, HJB),
                                       (520, 1100, 4, AC)])
@pytest.mark.parametrize("prec,tol", [(F.F64, 1e-10), (F.F32C, 1e-5)])
def test_warm_start(d, M, N, fam, prec, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hp, op = problems(d=d, M=M, N=N, prec=prec, seed=M, solver=F.SOLVER_CG, **fam)
    fixed, _ = problems(d=d, M=M, N=N, prec=prec, seed=M, solver=F.SOLVER_CG, cg_fixed_iters=400, **fam)
    x0 = workloads.points("normal_over_sqrt_d", 3, d, seed=d) * 0.3
    xt = torch.tensor(x0, device="cuda")
    print(f"[warm start] d={d} M={M} N={N} prec={prec}", flush=True)
    u, g, st = F.solve(hp, xt)
    ut, gt, stt = F.solve(hp, xt, tape=True)
    uf, gf, stf = F.solve(fixed, xt)
    torch.cuda.synchronize()
    assert torch.equal(u, ut) and torch.equal(g, gt) and torch.equal(u, uf) and torch.equal(g, gf)
    assert not st.any() and not stt.any() and not stf.any()
    for p in range(3):
        ref = OS.solve_point(op, x0[p], p)
        assert abs(float(u[p]) - ref["u"]) <= tol * abs(ref["u"]) and rel_err(g[p].cpu().numpy(), ref["grad"]) <= tol
