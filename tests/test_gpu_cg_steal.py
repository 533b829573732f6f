"""The CG loop's claims of items that nobody holds a ticket for.

* Few points whose chunks are no whole number of rounds over the resident blocks: 7 points take about what 8 take
  (blocks that waited out a part-empty round used to take other queues' items and to be away when their own came,
  which cost 2.6 times the time).
* All the work in one of 32 queues: 1024 points of which the 32 of queue 0 iterate and the others' right-hand sides are
  exactly zero (a saturated logistic under uniform weights of a power of two), so that the other queues' blocks have
  nothing of their own and claim queue 0's items.  Against the FP64 oracle.
"""
import time

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


@pytest.mark.parametrize("d,M,prec", [(3232, 1987, F.F64), (5544, 2965, F.F32C), (7485, 1137, F.F32C)])
def test_seven_points_take_no_longer_than_eight(d, M, prec):
    hp, _ = problems(d=d, M=M, N=2, prec=prec, seed=3, **AC)
    took = {}
    for P in (8, 7):
        x = torch.tensor(workloads.points("normal_over_sqrt_d", P, d, seed=1), device="cuda")
        ws = F.workspace(hp, P)
        ts = []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            _, _, st = F.solve(hp, x, ws=ws)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        assert not st.any()
        took[P] = min(ts)
    print(f"[cg steal] d={d} M={M}: 8 points {1e3 * took[8]:.1f} ms, 7 points {1e3 * took[7]:.1f}", flush=True)
    assert took[7] <= 1.3 * took[8]


def test_one_queue_with_all_the_work():
    d, M, P, N = 500, 4096, 1024, 2
    kw = dict(d=d, M=M, N=N, T=0.3, prec=F.F32C, seed=4, eps_h=0.0, f_kind=F.F_ZERO, g_kind=F.G_LOGISTIC, gp=(0.3, 0, 0, 0))
    hp, op = problems(gvec=np.full(d, 1.0 / np.sqrt(d)), **kw)
    x0 = np.full((P, d), 1e3)
    x0[::32] = workloads.points("normal_over_sqrt_d", 32, d, seed=5)
    print("[cg steal] one queue", flush=True)
    u, g, st = F.solve(hp, torch.tensor(x0, device="cuda"))
    torch.cuda.synchronize()
    u, g = u.cpu().numpy(), g.cpu().numpy()
    assert not st.cpu().numpy().any()
    idle = np.arange(P) % 32 != 0
    assert (u[idle] == 1.0).all() and not g[idle].any()
    for p in (0, 480, 992):
        ref = OS.solve_point(op, x0[p], p)
        assert abs(u[p] - ref["u"]) <= 1e-5 * abs(ref["u"]) and rel_err(g[p], ref["grad"]) <= 1e-5
