"""Workspace sizes of calls with many points (CPU: sizing only plans).  The chunk plan splits a point's rows for the CG
loop, and every chunk carries partial vectors and work items: calls of more points than the chip holds blocks ask for no
more than one chunk where more would not shorten them.  The bytes are those that the split into 4096 work items takes."""
import pytest

import paper_2510_02635_amd as F


@pytest.mark.parametrize("d,M,P,prec,solver,most", [
    (1000, 64, 65535, F.F64, F.SOLVER_AUTO, 38488715264), (100, 512, 16384, F.F64, F.SOLVER_CG, 8036880896),
    (200, 300, 8192, F.F32C, F.SOLVER_AUTO, 2451608064), (129, 300, 4096, F.F64, F.SOLVER_AUTO, 1519407616),
    (30, 17, 4000, F.F64, F.SOLVER_AUTO, 54644736)])
def test_many_points_ask_for_no_more(d, M, P, prec, solver, most):
    pb = F.Problem(d=d, M=M, N=3, T=0.3, prec=prec, solver=solver, f_kind=F.F_ALLEN_CAHN, fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC,
                   gp=(0.4, 0, 0, 0))
    assert F.workspace_size(pb, P) <= most
