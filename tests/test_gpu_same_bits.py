"""FP64, nearest-neighbour current: what a node gets does not depend on the sweep that serves it.  Bricks
against the march (a chunk length asked for selects it) and fitted tiles against 64 x 8 ones (which a long
chunk gives): u, B, J, alpha*, convexity and the positions after accepted steps, bit for bit; and the gradient
where the forward sweeps and their replay take fitted tiles.  (The sums are taken in another order, and the
FP32-mixed and octilateral sweeps leave the fusing of products to the compiler.)"""
import numpy as np
import pytest

import workloads as W
from gpu_util import banner, context, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _case(n, bc):
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.05 * min(g.h), seed=41)
    B0 = W.smooth_random_field(g, 0.6, seed=42) + np.array([0.2, -0.1, 1.0])[:, None, None, None]
    return g, x0, B0


def _choose(monkeypatch, tz):
    if tz is None:
        monkeypatch.delenv("RELAX_TZ", raising=False)
    else:
        monkeypatch.setenv("RELAX_TZ", str(tz))


# bricks / march: smallest, ragged, thin, every kind of face; fitted / 64 x 8: 32 x 16, 65 x 7, 37 x 13, 67 x 5, 34 x 15
CASES = [((4, 4, 4), (0, 0, 0), 9), ((5, 7, 9), (1, 0, 1), 2), ((17, 17, 17), (0, 0, 0), 5), ((200, 6, 5), (1, 1, 0), 9),
         ((6, 5, 300), (0, 1, 1), 9), ((41, 43, 47), (1, 1, 1), 6), ((64, 128, 64), (1, 0, 0), 9),
         ((96, 96, 96), (1, 1, 1), 24), ((129, 70, 70), (0, 0, 0), 24), ((73, 73, 120), (1, 1, 0), 24),
         ((67, 67, 203), (0, 0, 1), 24), ((34, 150, 130), (1, 0, 1), 24)]


@pytest.mark.parametrize("n,bc,tz", CASES, ids=[f"{c[0]}-{c[1]}" for c in CASES])
def test_a_node_has_the_same_bits_in_every_sweep(n, bc, tz, monkeypatch):
    g, x0, B0 = _case(n, bc)
    outs = []
    for chunk in (None, tz):
        _choose(monkeypatch, chunk)
        banner(f"bits {n} {bc} chunk {chunk}")
        with context(g, x0, B0, dt0=0.02 * min(g.h) ** 2, adaptive=True, tol=1e-7) as r:
            d = r.diagnostics()
            out = [r.velocity(), *r.fields(), *r.monitors()]
            steps = r.step(4)
            out = [host(t) for t in out] + [host(r.state()[0])]
        outs.append((out, [d[f] for f in ("min_det", "xi", "concave")],
                     [[s[f] for f in ("t", "dt", "Lambda", "xi", "min_det", "rejects")] for s in steps]))
    (a, da, sa), (b, db, sb) = outs
    for what, va, vb in zip(("u", "B", "J", "alpha", "kappa", "x"), a, b):
        assert np.array_equal(va, vb), (what, float(np.abs(va - vb).max()))
    assert da == db and sa == sb


GRADIENTS = [((96, 96, 96), (1, 1, 1)), ((129, 70, 70), (0, 0, 0)), ((73, 73, 120), (0, 1, 0)), ((67, 67, 203), (1, 0, 1))]


@pytest.mark.parametrize("n,bc", GRADIENTS, ids=[f"{c[0]}-{c[1]}" for c in GRADIENTS])
def test_gradient_through_fitted_tiles(n, bc, monkeypatch):
    """The replay stores y_4 and y_6 from fitted tiles; the reverse sweeps have 64 x 8 tiles of their own,
    whose results do not depend on the chunk length.  The R2 seed takes u from the diagnostics sweep."""
    g, x0, B0 = _case(n, bc)
    outs = []
    for chunk in (None, 24):
        _choose(monkeypatch, chunk)
        banner(f"gradient bits {n} {bc} chunk {chunk}")
        with context(g, x0, B0, K_record=3, dt0=0.02 * min(g.h) ** 2, adaptive=False, record=True,
                     checkpoint_every=2) as r:
            r.step(3, diag=False)
            outs.append([host(t) for t in r.backward(1.0, 0.3)])
    for a, b in zip(*outs):
        assert np.isfinite(a).all() and np.abs(a).max() > 0.0
        assert np.array_equal(a, b)
