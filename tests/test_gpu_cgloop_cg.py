"""The device-side CG loop with the CG on every level (SOLVER_CG), over the depths of its arrival tree: shapes whose
d <= 128 the direct solves would otherwise take.  Against the FP64 oracle and the host-polled loop
(FBSDE_CG_HOST_LOOP=1), with iteration counts that are never zero; the streamed-row record against those counts; and a
captured graph of such a solve over several replays.
"""
import os

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import scheme as OS  # noqa: E402
from paper_2510_02635_amd import workloads  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

AC = dict(f_kind=F.F_ALLEN_CAHN, fp=(1.0, 1.0, 0, 0), g_kind=F.G_AC, gp=(0.4, 0, 0, 0), T=0.3, solver=F.SOLVER_CG)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F.autotune_reset()


# (d, M, N, P, prec, tol); up to 32 points a chunk is 16 rows at least and an item per resident block at most
SHAPES = [
    (100, 1024, 3, 4096, F.F64, 1e-10),       # one chunk per point: the chunk's block does the CG step; warm levels
    (30, 100, 3, 5, F.F64, 1e-10),            # 6 chunks: one tree level, part-filled
    (100, 512, 4, 3, F.F64, 1e-10),           # 32 chunks: two levels
    (200, 384, 3, 4, F.F64, 1e-10),           # 24 chunks: two levels, part-filled
    (100, 1040, 2, 1, F.F64, 1e-10),          # 65 chunks: three levels, the last ones of one child
    (100, 8192, 2, 1, F.F64, 1e-10),          # 512 chunks: three levels, full
    (64, 2048, 3, 6, F.F32C, 1e-5),           # 128 chunks, FP32C, warm levels
    (120, 110, 3, 40, F.F32C, 1e-5),          # rank-deficient: FP64 arithmetic on the FP32 state; two points a queue
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"d{s[0]}_M{s[1]}_P{s[3]}_{'f64' if s[4] == F.F64 else 'f32c'}" for s in SHAPES])
def test_cg_on_every_level(shape):
    d, M, N, P, prec, tol = shape
    hp, op = problems(d=d, M=M, N=N, seed=3, instance=2, prec=prec, **AC)
    x0 = workloads.points("normal:0.4", P, d, seed=d + M)
    xt = torch.tensor(x0, device="cuda")
    print(f"[cgloop cg] d={d} M={M} P={P} prec={prec}", flush=True)
    u, g, st, it = F.solve(hp, xt, return_iters=True)
    torch.cuda.synchronize()
    os.environ["FBSDE_CG_HOST_LOOP"] = "1"
    try:
        uh, gh, sth, ith = F.solve(hp, xt, return_iters=True)
        torch.cuda.synchronize()
    finally:
        os.environ.pop("FBSDE_CG_HOST_LOOP")
    assert min(it) > 0 and min(ith) > 0 and not st.any() and not sth.any()
    # the loops sum more than four chunks in different orders, which can move a stopping test by one iteration
    assert all(abs(a - b) <= 1 for a, b in zip(it, ith))
    assert rel_err(u.cpu().numpy(), uh.cpu().numpy()) <= (1e-13 if prec == F.F64 else 1e-6)
    assert rel_err(g.cpu().numpy(), gh.cpu().numpy()) <= (1e-11 if prec == F.F64 else 1e-5)
    for p in sorted({0, P - 1}):
        ref = OS.solve_point(op, x0[p], p)
        assert abs(u[p].item() - ref["u"]) <= tol * abs(ref["u"]) and rel_err(g[p].cpu().numpy(), ref["grad"]) <= tol


def test_streamed_rows_are_the_iterations():
    d, M = 50, 700
    hp, _ = problems(d=d, M=M, N=4, seed=1, **AC)
    ws = F.workspace(hp, 1)
    _, _, st, it = F.solve(hp, torch.tensor(workloads.points("normal:0.5", 1, d, seed=2), device="cuda"), ws=ws,
                           return_iters=True)
    rows = F.workspace_cg_rows(ws)
    assert not st.any() and rows > 0 and rows == M * sum(it)


def test_graph_of_cg_levels():
    d, M, P = 100, 512, 2
    hp, op = problems(d=d, M=M, N=5, seed=0, **AC)
    x0 = workloads.points("normal:0.3", P, d, seed=4)
    xt = torch.tensor(x0, device="cuda")
    u0, g0, _, it = F.solve(hp, xt, return_iters=True)
    torch.cuda.synchronize()
    assert min(it) > 0
    cs = F.CapturedSolve(hp, xt)
    for _ in range(3):
        u, g, st = cs.launch()
        torch.cuda.synchronize()
        assert torch.equal(u, u0) and torch.equal(g, g0) and not st.any()
        torch.zeros(1024, device="cuda").sum().item()   # eager work between replays
    ref = OS.solve_point(op, x0[0], 0)
    assert abs(u0[0].item() - ref["u"]) <= 1e-10 * abs(ref["u"])
