"""relax_backward in the middle of a run leaves the run as it was: its replay shares the stage vectors with
the forward steps.  Positions, step records and the gradient at the end, bit for bit, on bricks and on the
march, with fixed steps and with rejected attempts."""
import numpy as np
import pytest

import workloads as W
from gpu_util import banner, context, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("tz", [None, 5])
@pytest.mark.parametrize("kw", [dict(dt0=1e-4, adaptive=False), dict(dt0=3e-2, adaptive=True, tol=1e-8)],
                         ids=["fixed", "adaptive"])
def test_backward_between_steps(kw, tz, monkeypatch):
    banner(f"backward between steps {kw} chunk {tz}")
    if tz is not None:
        monkeypatch.setenv("RELAX_TZ", str(tz))
    n, bc = (18, 21, 14), (0, 1, 0)
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.02 * min(g.h), seed=51)
    B0 = W.smooth_random_field(g, 0.6, seed=52) + np.array([0.2, -0.1, 1.0])[:, None, None, None]
    outs = []
    for between in (False, True):
        with context(g, x0, B0, K_record=6, record=True, checkpoint_every=2, **kw) as r:
            steps = r.step(3)
            if between:
                r.backward(0.7, 0.2)
            steps += r.step(3)
            x = host(r.state()[0])
            outs.append((steps, x, [host(t) for t in r.backward(1.0, 0.3)]))
    (sa, xa, ga), (sb, xb, gb) = outs
    if kw["adaptive"]:
        assert sum(s["rejects"] for s in sa) > 0
    assert sa == sb and np.array_equal(xa, xb)
    for a, b in zip(ga, gb):
        assert np.array_equal(a, b)
