"""Workspaces below the plan's own size: calls keep the sizes that earlier kernels asked for.

* The direct dual solve, whose M x M matrices are laid out without padding and over the CG's buffers: within the fixed
  array of the allocation-free entry point, and in P M (M + 1) doubles beyond a workspace without any CG buffer to lie
  over (cg_maxit = 1, one chunk a point).
* Its results there against the FP64 oracle (1e-10), with no CG iteration.
* Every other entry point with room for fewer partial vectors than the plan takes: x-dependent coefficients and a
  diffusion matrix, forward and reverse (the reverse mode also in the larger buffer that the small workspace is a part
  of), the autotuner, graphs, and the tiled batched schedule; against the same call in a workspace of the plan's size, to
  the FP64 tolerance 1e-10, since the sums are split differently.
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


D, M, P, N = 1100, 600, 3, 2          # 37 chunks a point planned, nine in a smaller workspace
LESS = 20 * P * D * 8                 # room for 20 partial vectors fewer a point
COEF = (0.05, 0.2, 0.1, 0.6)


def _near(a, b):
    torch.cuda.synchronize()
    assert rel_err(a.cpu().numpy(), b.cpu().numpy()) <= 1e-10


def _case():
    hp, _ = problems(d=D, M=M, N=N, seed=1, **AC)
    return hp, torch.tensor(workloads.points("normal_over_sqrt_d", P, D, seed=2), device="cuda")


def test_coefficient_family_and_its_reverse_mode():
    hp, x = _case()
    ub = torch.ones(P, dtype=torch.float64, device="cuda")
    full = F.coef_workspace_size(hp, P, *COEF, tape=True)
    out = []
    for fwd, bwd in ((full, full), (full - LESS, full - LESS), (full - LESS, full)):
        buf = _bytes(full)
        u, g, st = F.solve_coef(hp, x, *COEF, ws=buf[:fwd], tape=True)
        xb, gpb, fpb, st2 = F.solve_coef_backward(hp, x, ub, buf[:bwd], *COEF)
        torch.cuda.synchronize()
        assert not st.any() and not st2.any()
        out.append((u, g, xb, gpb, fpb))
    for o in out[1:]:
        for a, b in zip(o, out[0]):
            _near(a, b)
    u, g, st = F.solve_coef(hp, x, *COEF, ws=_bytes(F.coef_workspace_size(hp, P, *COEF) - LESS))
    _near(u, out[0][0])
    with pytest.raises(F.FbsdeError):
        F.solve_coef(hp, x, *COEF, ws=_bytes(F.coef_workspace_size(hp, P, *COEF) - 6 * LESS))


def test_diffusion_matrix_and_its_reverse_mode():
    hp, x = _case()
    sg = torch.eye(D, dtype=torch.float64, device="cuda") * 1.2
    sg[0, D - 1] = 0.3
    ub = torch.ones(P, dtype=torch.float64, device="cuda")
    full = F.sigma_workspace_size(hp, P, tape=True)
    out = []
    for fwd, bwd in ((full, full), (full - LESS, full - LESS), (full - LESS, full)):
        buf = _bytes(full)
        u, g, st = F.solve_sigma(hp, x, sg, ws=buf[:fwd], tape=True)
        r = F.solve_sigma_backward(hp, x, sg, ub, buf[:bwd])
        torch.cuda.synchronize()
        assert not st.any()
        out.append((u, g, *r[:3]))
    for o in out[1:]:
        for a, b in zip(o, out[0]):
            _near(a, b)
    with pytest.raises(F.FbsdeError):
        F.solve_sigma(hp, x, sg, ws=_bytes(F.sigma_workspace_size(hp, P) - 6 * LESS))


def test_autotuner_and_graph():
    import ctypes
    from paper_2510_02635_amd import _native as NV
    hp, x = _case()
    F.autotune_reset()
    u0, g0, _ = F.solve(hp, x)
    small = _bytes(F.workspace_size(hp, P) - LESS)
    u, g = torch.empty_like(u0), torch.empty_like(g0)
    st = torch.empty(P, dtype=torch.int32, device="cuda")
    h = ctypes.c_void_p()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    NV.check(NV.load().fbsde_graph_capture(ctypes.byref(hp.c()), P, x.data_ptr(), u.data_ptr(), g.data_ptr(), st.data_ptr(),
                                           small.data_ptr(), small.numel(), 0, ctypes.byref(h), stream))
    for _ in range(3):
        u.zero_()
        NV.check(NV.load().fbsde_graph_launch(h, stream))
        _near(u, u0)
        _near(g, g0)
        assert not st.any()
    NV.check(NV.load().fbsde_graph_destroy(h))
    F.autotune(hp, x, ws=small)
    try:
        u, g, st = F.solve(hp, x, ws=small)
        _near(u, u0)
        _near(g, g0)
    finally:
        F.autotune_reset()


def test_tiled_batch():
    import ctypes
    from paper_2510_02635_amd import _native as NV, api
    hp, x = _case()
    h2, _ = problems(d=90, M=700, N=N, seed=2, instance=1, **AC)
    pbs, xs = [hp, h2, hp], [x, x[:, :90].contiguous(), x]
    n, cps, Ps = api._batch_common(pbs, xs)
    opts = api._batch_opts("tiled", 3, 0, 512)
    Pv, ov, stream = ctypes.cast(Ps, ctypes.c_void_p), ctypes.byref(opts), api._stream()
    ubs = [torch.ones(P, dtype=torch.float64, device="cuda")] * 3

    def call(ws, adjoint):
        us = [torch.empty(P, dtype=torch.float64, device="cuda") for _ in pbs]
        gs = [torch.empty_like(v) for v in xs]
        sts = [torch.empty(P, dtype=torch.int32, device="cuda") for _ in pbs]
        if not adjoint:
            NV.check(NV.load().fbsde_solve_batched(cps, n, Pv, api._ptrs(xs), api._ptrs(us),
                                                   ctypes.cast(api._ptrs(gs), ctypes.c_void_p), api._ptrs(sts), ov,
                                                   ws.data_ptr(), ws.numel(), stream))
        else:
            gps, fps = ([torch.empty(4, dtype=torch.float64, device="cuda") for _ in pbs] for _ in range(2))
            NV.check(NV.load().fbsde_solve_batched_backward(cps, n, Pv, api._ptrs(xs), api._ptrs(ubs), api._ptrs(us),
                                                            api._ptrs(gs), api._ptrs(gps), api._ptrs(fps), api._ptrs(sts),
                                                            ov, ws.data_ptr(), ws.numel(), stream))
        torch.cuda.synchronize()
        assert not any(bool(s.any()) for s in sts)
        return us + gs

    for adjoint in (False, True):
        full = F.batched_workspace(pbs, xs, adjoint=adjoint).numel()
        for a, b in zip(call(_bytes(full - 3 * LESS), adjoint), call(_bytes(full), adjoint)):
            _near(a, b)
        with pytest.raises(F.FbsdeError):
            call(_bytes(full - 25 * LESS), adjoint)
