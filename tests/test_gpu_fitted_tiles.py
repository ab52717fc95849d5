"""The z-march on tiles that are not 64 x 8 (grids whose extents 64 x 8 tiles would cover with many idle
threads), against the oracle: tiles of 65 x 7 (threads without a node), 34 x 15 and 37 x 13 (waves over
several rows, rows off cache lines), 32 x 16, 49 x 10, and with the octilateral current 50 x 10.  One
evaluation and one fixed step, with the bounds of one evaluation (1e-12 normwise; B 1e-13; FP32-mixed
increment 2e-5 as everywhere)."""
import numpy as np
import pytest

import oracle
import paper_1405_0942_amd as R
import workloads as W
from gpu_util import banner, context, host, nrel, nrel_inc, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

FP64, MIXED, NNN = dict(), dict(precision=R.RELAX_FP32_MIXED), dict(curl=R.RELAX_CURL_NNN)
CASES = [((129, 70, 70), (0, 0, 0), FP64), ((34, 150, 130), (1, 0, 1), FP64), ((73, 73, 120), (1, 1, 0), MIXED),
         ((96, 96, 96), (1, 1, 1), FP64), ((193, 60, 60), (0, 1, 0), MIXED), ((150, 100, 70), (0, 0, 1), NNN)]


@pytest.mark.parametrize("n,bc,kw", CASES, ids=[f"{c[0]}-{c[1]}-{i}" for i, c in enumerate(CASES)])
def test_fitted_tiles_match_the_oracle(n, bc, kw):
    banner(f"fitted tiles {n} {bc} {kw}")
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.02 * min(g.h), seed=31)
    B0 = W.smooth_random_field(g, 0.6, seed=32) + np.array([0.2, -0.1, 1.0])[:, None, None, None]
    dt = 0.02 * min(g.h) ** 2
    with context(g, x0, B0, dt0=dt, adaptive=False, **kw) as r:
        d = r.diagnostics()
        u = host(r.velocity())
        B, J = (host(t) for t in r.fields())
        r.step(1)
        x1 = host(r.state()[0])
    with oracle.curl(oracle.CURL_NNN if kw is NNN else oracle.CURL_NN):
        o = oracle.fields(g, x0, B0)
        od = oracle.diagnostics(g, x0, B0, oracle.null_threshold(B0))
        o1 = oracle.run(g, x0, B0, 1, dt=dt, mode=oracle.MODE_FIXED)
    assert nrel(B, o["B"]) < 1e-13 and nrel(J, o["J"]) < 1e-12 and nrel(u, o["u"]) < 1e-12
    assert d["concave"] == oracle.convexity(g, x0)[1]
    assert rel(d["E_M"], od["E_M"]) < 1e-12 and rel(d["min_det"], od["min_det"]) < 1e-13
    assert rel(d["R2"], od["R2"]) < 1e-11 and rel(d["xi"], od["xi"]) < 1e-11
    assert nrel_inc(x1, x0, o1["x"]) < (2e-5 if kw is MIXED else 1e-11)
