"""The small-grid sweeps (brick.hip) against the z-marching ones (stage.hip) on the same inputs, at the
sizes where a brick can go wrong: the smallest grids, bricks that do not divide the grid, thin and long
grids, every boundary mix, and both sides of the size at which the march takes over.

Both evaluate the same operations per node; a compiler may contract them differently, which is worth an
ulp or two per operation, so the bounds are those of one evaluation against the oracle (1e-13 for B,
1e-12 for J, u and an increment; FP32-mixed increments 2e-6, 16 ulps of FP32)."""
import numpy as np
import pytest

import paper_1405_0942_amd as R
import workloads as W
from gpu_util import banner, context, host, nrel, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

FP64, MIXED = dict(), dict(precision=R.RELAX_FP32_MIXED)
NNN = dict(curl=R.RELAX_CURL_NNN)
CASES = [
    ((4, 4, 4), (0, 0, 0), FP64), ((4, 4, 4), (1, 1, 1), NNN), ((5, 7, 9), (1, 0, 1), MIXED),
    ((17, 17, 17), (0, 0, 0), FP64), ((13, 29, 11), (0, 1, 1), NNN), ((33, 33, 33), (0, 0, 0), MIXED),
    ((200, 6, 5), (1, 1, 0), FP64), ((6, 5, 300), (0, 1, 1), FP64), ((5, 211, 7), (1, 0, 0), NNN),
    ((41, 43, 47), (1, 1, 1), FP64), ((41, 43, 47), (0, 0, 1), NNN),
    ((64, 128, 64), (1, 0, 0), FP64),  # 2^19 nodes: the largest grids that take bricks
    ((84, 84, 85), (0, 1, 0), FP64),  # 599 760 nodes: the march, short chunks against the chosen ones
]


@pytest.mark.parametrize("n,bc,kw", CASES, ids=[f"{c[0]}-{c[1]}-{i}" for i, c in enumerate(CASES)])
def test_bricks_match_the_march(n, bc, kw, monkeypatch):
    banner(f"bricks {n} {bc} {kw}")
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.02 * min(g.h), seed=11)
    B0 = W.smooth_random_field(g, 0.6, seed=12) + np.array([0.2, -0.1, 1.0])[:, None, None, None]
    outs = []
    for tz in (None, "9"):
        if tz is None:
            monkeypatch.delenv("RELAX_TZ", raising=False)
        else:
            monkeypatch.setenv("RELAX_TZ", tz)  # a chunk length selects the march
        with context(g, x0, B0, dt0=0.02 * min(g.h) ** 2, adaptive=False, **kw) as r:
            d = r.diagnostics()
            u = host(r.velocity())
            B, J = (host(t) for t in r.fields())
            kappa = host(r.monitors()[1])
            r.step(2)
            outs.append((u, B, J, kappa, host(r.state()[0]) - x0, d))
    (u, B, J, kappa, dx, d), (um, Bm, Jm, km, dxm, dm) = outs
    assert np.array_equal(kappa, km) and d["concave"] == dm["concave"]
    assert nrel(B, Bm) < 1e-13 and nrel(J, Jm) < 1e-12 and nrel(u, um) < 1e-12
    # the increment up to the rounding of the stored positions
    ulp = np.spacing(np.abs(x0).max())
    assert np.abs(dx - dxm).max() <= (2e-6 if kw is MIXED else 1e-12) * np.abs(dxm).max() + 2 * ulp
    for f in ("E_M", "xi", "R2", "min_det"):
        assert rel(d[f], dm[f]) < 1e-12


GRAD_CASES = [((4, 4, 4), (0, 0, 0)), ((5, 6, 7), (1, 1, 1)), ((17, 17, 17), (0, 0, 0)), ((70, 11, 9), (0, 1, 0)),
              ((7, 66, 13), (1, 0, 1)), ((41, 43, 47), (0, 0, 1))]


@pytest.mark.parametrize("n,bc", GRAD_CASES, ids=[f"{c[0]}-{c[1]}" for c in GRAD_CASES])
def test_gradient_bricks_match_the_march(n, bc, monkeypatch):
    """Both orders of the same sums: 1e-12 normwise, as against the oracle's complex step (1e-10)."""
    banner(f"gradient bricks {n} {bc}")
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.02 * min(g.h), seed=21)
    B0 = W.smooth_random_field(g, 0.6, seed=22) + np.array([0.2, -0.1, 1.0])[:, None, None, None]
    outs = []
    for tz in (None, "9"):
        if tz is None:
            monkeypatch.delenv("RELAX_TZ", raising=False)
        else:
            monkeypatch.setenv("RELAX_TZ", tz)
        with context(g, x0, B0, K_record=3, dt0=0.02 * min(g.h) ** 2, adaptive=False, record=True,
                     checkpoint_every=2) as r:
            r.step(3, diag=False)
            outs.append([host(t) for t in r.backward(1.0, 0.3)])
    for a, b in zip(*outs):
        assert nrel(a, b) < 1e-12
