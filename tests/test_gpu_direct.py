"""The direct level solves (csrc/fbsde_direct.hpp): primal (M > d + 1, d <= 128) and dual (M <= 128), at system
sizes around the edges of the 16 x 16 tiles and of the blocks of four pivots, one and many slices of the Gram
matrix, both precisions, and a workspace that holds no slices.  The oracle solves the same systems by a library
Cholesky in FP64; the tolerances are the precision modes' (1e-10 FP64, 1e-5 FP32C).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402
from paper_2510_02635_amd import workloads  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

DEV = "cuda"
HJB = dict(f_kind=F.F_HJB, fp=(0.8, 0, 0, 0), g_kind=F.G_HJB_LOG, gp=(1.0, 0, 0, 0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F._native.load()


# (d, M, P, prec, tol): primal where M > d + 1, dual otherwise
DIRECT = [(1, 40, 3, F.F64, 1e-10), (3, 60, 2, F.F64, 1e-10), (4, 16, 2, F.F64, 1e-10), (15, 33, 2, F.F64, 1e-10),
          (16, 64, 2, F.F64, 1e-10), (17, 65, 2, F.F64, 1e-10), (47, 200, 2, F.F64, 1e-10), (48, 201, 2, F.F64, 1e-10),
          (64, 129, 2, F.F64, 1e-10), (96, 300, 600, F.F64, 1e-10), (127, 260, 2, F.F64, 1e-10),
          (128, 2000, 1, F.F64, 1e-10), (128, 300, 2, F.F32C, 1e-5), (33, 100, 520, F.F32C, 1e-5),
          (100, 16, 2, F.F64, 1e-10), (127, 112, 2, F.F64, 1e-10), (130, 128, 520, F.F64, 1e-10),
          (128, 64, 2, F.F32C, 1e-5)]


@pytest.mark.parametrize("case", DIRECT, ids=[f"d{c[0]}_M{c[1]}_P{c[2]}_{c[3]}" for c in DIRECT])
def test_direct_level_solve_sizes(case):
    d, M, P, prec, tol = case
    hp, op = problems(d=d, M=M, N=3, T=0.3, prec=prec, seed=d, instance=M, **HJB)
    x0 = workloads.points("normal_over_sqrt_d", P, d, seed=M)
    print(f"[direct] d={d} M={M} P={P} prec={prec}", flush=True)
    u, g, st, it = F.solve(hp, torch.tensor(x0, device=DEV), return_iters=True)
    torch.cuda.synchronize()
    u, g = u.cpu().numpy(), g.cpu().numpy()
    assert it == [0, 0, 0] and not st.any()
    for p in sorted({0, P - 1}):
        ref = OS.solve_point(op, x0[p], p)
        assert abs(u[p] - ref["u"]) <= tol * abs(ref["u"]) and rel_err(g[p], ref["grad"]) <= tol


def test_direct_solve_keeps_to_its_rule():
    # beyond d = 128, with a cap below d, without a ridge or with SOLVER_CG the level stays with the CG
    for kw in (dict(d=129, M=300), dict(d=40, M=100, cg_maxit=39), dict(d=20, M=60, ridge_rel=0.0),
               dict(d=20, M=60, solver=F.SOLVER_CG)):
        hp, _ = problems(N=2, T=0.3, seed=1, **HJB, **kw)
        x = torch.tensor(workloads.points("normal_over_sqrt_d", 2, kw["d"], 4), device=DEV)
        assert min(F.solve(hp, x, return_iters=True)[3]) > 0


def test_direct_solve_in_a_workspace_without_room_for_its_slices():
    # the CG's workspace holds no partial Gram matrices: fewer slices, or the CG, and the same result
    d, M, P = 90, 700, 3
    hp, op = problems(d=d, M=M, N=3, T=0.3, seed=2, **HJB)
    hc, _ = problems(d=d, M=M, N=3, T=0.3, seed=2, solver=F.SOLVER_CG, **HJB)
    x0 = workloads.points("normal_over_sqrt_d", P, d, 5)
    xt = torch.tensor(x0, device=DEV)
    small, full = F.workspace_size(hc, P), F.workspace_size(hp, P)
    assert small < full
    ref = OS.solve_point(op, x0[1], 1)
    for size in (small, (small + full) // 2, full):
        u, g, st = F.solve(hp, xt, ws=torch.empty(size, dtype=torch.uint8, device=DEV))
        torch.cuda.synchronize()
        assert not st.any() and abs(u[1].item() - ref["u"]) <= 1e-10 * abs(ref["u"])
        assert rel_err(g[1].cpu().numpy(), ref["grad"]) <= 1e-10
    with pytest.raises(F.FbsdeError):
        F.solve(hp, xt, ws=torch.empty(small - 256, dtype=torch.uint8, device=DEV))
