"""The register-resident factorisation (csrc/fbsde_spd.hpp) on systems far from one: sigma of 1e+-80 and 1e+-100 gives
matrices of 1e+-160 and 1e+-200 (the anchors: 2e77 and 8e77, beyond which |Z|^2 leaves the range), inside FP64's range while a product of two pivots is not.  Direct primal and dual
solves and the literal anchors, against the FP64 oracle at the schemes' tolerances (1e-10; |Z|^2 and sum Z 1e-8).  For
a tiny sigma every particle sits at x0 to rounding, so u is compared and the slope, rounding over the ridge, only has to
be finite.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import paper_2510_02635_amd as F  # noqa: E402
from oracle import literal as OL  # noqa: E402
from oracle import scheme as OS  # noqa: E402

from _convert import problems, rel_err  # noqa: E402

HJB = dict(f_kind=F.F_HJB, fp=(1.0, 0, 0, 0), g_kind=F.G_HJB_LOG, gp=(1.0, 0, 0, 0), T=0.3)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("d,M,s", [(10, 40, 1e-100), (10, 8, 1e-100), (10, 40, 1e-80), (10, 8, 1e-80), (100, 300, 1e-80),
                                   (100, 90, 1e-80), (10, 40, 1e80), (10, 8, 1e80), (100, 300, 1e80), (100, 90, 1e80),
                                   (10, 40, 1e100), (10, 8, 1e100), (100, 300, 1e100), (100, 90, 1e100)])
def test_direct_solves_of_far_scaled_systems(d, M, s):
    hp, op = problems(d=d, M=M, N=3, s=s, seed=1, **HJB)
    x0 = 0.1 * np.random.default_rng(d).normal(size=(2, d))
    u, g, st, it = F.solve(hp, torch.tensor(x0, device="cuda"), return_iters=True)
    torch.cuda.synchronize()
    u, g = u.cpu().numpy(), g.cpu().numpy()
    assert it == [0, 0, 0] and not st.any() and np.isfinite(g).all()
    for p in range(2):
        ref = OS.solve_point(op, x0[p], p)
        assert abs(u[p] - ref["u"]) <= 1e-10 * abs(ref["u"])
        if s > 1.0:
            assert rel_err(g[p] * s, ref["grad"] * s) <= 1e-10


@pytest.mark.parametrize("s", [2e77, 8e77])
@pytest.mark.parametrize("M", [12, 50])
def test_literal_anchors_of_far_scaled_systems(M, s):
    hp, op = problems(d=4 * M, M=M, N=2, s=s, seed=M, ridge_rel=1e-2, **HJB)
    x0 = 0.1 * np.random.default_rng(M).normal(size=(2, 4 * M))
    u, st, Y, zs = F.solve_literal(hp, torch.tensor(x0, device="cuda"), k_stop=1, want_Y=True, want_zstats=True)
    torch.cuda.synchronize()
    u, st, Y, zs = (t.cpu().numpy() for t in (u, st, Y, zs))
    assert not st.any()
    for p in range(2):
        ref = OL.solve_point(op, x0[p], p, k_stop=1, tape=True)
        assert abs(u[p] - ref["u"]) <= 1e-10 * max(1.0, abs(ref["u"]))
        assert np.max(np.abs(Y[p] - ref["Y"])) <= 1e-10 * max(1.0, np.max(np.abs(ref["Y"])))
        for e, r in ((0, ref["zz"][1]), (1, ref["zs"][1])):
            assert np.max(np.abs(zs[p, :, e] - r)) <= 1e-8 * np.max(np.abs(r))
