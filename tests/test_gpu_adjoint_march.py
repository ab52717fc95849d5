"""The z-marching reverse sweeps (adjoint.hip) against the brick ones on the same inputs, at the sizes
where a march can go wrong: tiles with idle columns and rows, tiles that wrap onto themselves, one to
several tiles across, chunks of one plane up, every kind of face.

Both evaluate the same sums with at most some 300 roundings per value and sweep; 3 steps are 18 sweeps,
and the differences of neighbouring values lose about one digit: 18 * 300 * 1.1e-16 * 10 = 6e-12."""
import numpy as np
import pytest

import paper_1405_0942_amd as R
import workloads as W
from gpu_util import banner, dev, host, nrel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

CASES = [
    ((4, 4, 4), (0, 0, 0), 1), ((4, 4, 4), (1, 1, 1), 4), ((64, 8, 8), (1, 1, 0), 3), ((66, 9, 7), (1, 0, 1), 7),
    ((63, 17, 9), (0, 1, 0), 2), ((130, 5, 6), (0, 0, 1), 5), ((129, 16, 12), (1, 1, 1), 12),
    ((65, 25, 10), (0, 0, 0), 4),
]


@pytest.mark.parametrize("n,bc,tz", CASES, ids=[f"{c[0]}-{c[1]}-{c[2]}" for c in CASES])
def test_reverse_march_matches_bricks(n, bc, tz, monkeypatch):
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.02 * min(g.h), seed=21)
    B0 = W.smooth_random_field(g, 0.6, seed=22) + np.array([0.2, -0.1, 1.0])[:, None, None, None]
    cfg = R.make_config(g, dt0=1e-4, adaptive=False, record=True, checkpoint_every=2)
    grads = []
    for chunk in (None, str(tz)):
        if chunk is None:
            monkeypatch.delenv("RELAX_TZ", raising=False)
        else:
            monkeypatch.setenv("RELAX_TZ", chunk)
        for seeds in ((1.0, 0.0), (0.3, 1.0)):
            banner(f"reverse sweeps {n} {bc} tz {chunk} seeds {seeds}")
            with R.Relaxation(cfg, dev(x0), dev(B0), K_record=3) as r:
                r.step(3, diag=False)
                grads.append([host(v) for v in r.backward(*seeds)])
    for brick, march in zip(grads[:2], grads[2:]):
        for b, m in zip(brick, march):
            assert np.isfinite(m).all()
            assert nrel(m, b) <= 6e-12
