"""The register-resident solve of small symmetric positive definite systems (csrc/fbsde_spd.hpp) at the edges of
its 16 x 16 tiles and of its blocks of four pivots, through the paper-literal anchors: M x M systems around
every multiple of 16 (the right-hand side's column starts a tile of its own there) and of 4 (padding rows).
The oracle solves the same systems by a library factorisation; the tolerances are the literal scheme's (1e-10,
|Z|^2 and sum Z 1e-8).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import literal as OL  # noqa: E402

from _convert import problems  # noqa: E402

DEV = "cuda"
HJB = dict(f_kind=F.F_HJB, fp=(0.8, 0, 0, 0), g_kind=F.G_HJB_LOG, gp=(1.0, 0, 0, 0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F._native.load()


@pytest.mark.parametrize("M", [3, 4, 5, 12, 13, 15, 17, 31, 32, 33, 47, 48, 49, 64, 65, 96, 97, 127, 128, 129, 145, 160,
                               176, 192, 208, 209, 240, 252, 253])
def test_literal_anchor_tile_edges(M):
    hp, op = problems(d=20, M=M, N=2, T=0.4, seed=M, ridge_rel=1e-2, **HJB)
    x0 = 0.3 * np.random.default_rng(M).normal(size=(2, 20))
    print(f"[spd literal] M={M}", flush=True)
    u, st, Y, zs = F.solve_literal(hp, torch.tensor(x0, device=DEV), k_stop=1, want_Y=True, want_zstats=True)
    torch.cuda.synchronize()
    u, st, Y, zs = (t.cpu().numpy() for t in (u, st, Y, zs))
    assert not st.any()
    for p in range(2):
        ref = OL.solve_point(op, x0[p], p, k_stop=1, tape=True)
        assert abs(u[p] - ref["u"]) <= 1e-10 * max(1.0, abs(ref["u"]))
        assert np.max(np.abs(Y[p] - ref["Y"])) <= 1e-10 * max(1.0, np.max(np.abs(ref["Y"])))
        for e, r in ((0, ref["zz"][1]), (1, ref["zs"][1])):
            assert np.max(np.abs(zs[p, :, e] - r)) <= 1e-8 * np.max(np.abs(r))
