"""The timed moments pass is the one that the solve's levels run: on a rank-deficient design in FP32C it sums in FP64 on
the FP32 state.  Its partial sums are looked for in the workspace it leaves: sum_j w_j W_j over the rows of the first
chunk, to 1e-13 (FP32 products would be 1e-8 off)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402


@pytest.mark.parametrize("d,M", [(80, 70), (300, 200)])
def test_moments_sum_as_the_solve_does(d, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pb = F.Problem(d=d, M=M, N=1, T=0.3, prec=F.F32C, solver=F.SOLVER_CG, eps_h=0.0, f_kind=F.F_ALLEN_CAHN,
                   fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC, gp=(0.4, 0, 0, 0), seed=2)
    x = torch.zeros((1, d), dtype=torch.float64, device="cuda")
    ws = torch.zeros(F.workspace_size(pb, 1), dtype=torch.uint8, device="cuda")
    F.solve(pb, x, ws=ws)                       # one level: the state stays at t_1
    F.time_kernel(pb, 1, "moments", ws, reps=2)
    W = F.terminal(pb, x)[0][0, :, :d].double()
    torch.cuda.synchronize()
    buf = ws.view(torch.float64)
    found = False
    for rows in range(1, M):                    # not all: the solve leaves the mean of all rows too
        want = W[:rows].sum(0) / M
        for at in ((buf - want[0]).abs() <= 1e-13 * want[0].abs()).nonzero().flatten().tolist():
            got = buf[at:at + d]
            found |= got.numel() == d and bool(((got - want).abs() <= 1e-13 * want.abs().max()).all())
    assert found
