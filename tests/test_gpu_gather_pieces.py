"""A gather of the reverse pass launched in pieces (grids of more workgroups than one launch holds; the
64 x 4 build takes 64 a launch) gives the gradient of one launch, bit for bit: 54, 297 and 153 workgroups."""
import numpy as np
import pytest

import paper_1405_0942_amd as R
from paper_1405_0942_amd import build as B
import workloads as W
from gpu_util import banner, context, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("n,bc", [((70, 11, 9), (0, 1, 0)), ((33, 33, 33), (0, 0, 0)), ((9, 66, 9), (1, 0, 1))])
def test_pieces_of_a_gather_make_the_whole(n, bc):
    g = W.make_grid(n, [(0.0, 0.1 * v) for v in n], bc)
    x0 = W.distorted_grid(g, 0.02 * min(g.h), seed=21)
    B0 = W.smooth_random_field(g, 0.6, seed=22) + np.array([0.2, -0.1, 1.0])[:, None, None, None]

    def gradient():
        with context(g, x0, B0, K_record=3, dt0=1e-4, adaptive=False, record=True, checkpoint_every=2) as r:
            r.step(3, diag=False)
            return [host(t) for t in r.backward(1.0, 0.3)]

    banner(f"gather {n} in one launch")
    whole = gradient()
    banner(f"gather {n} in pieces")
    with R.using_library(B.LIB_TY4):
        pieces = gradient()
    for a, b in zip(whole, pieces):
        assert np.array_equal(a, b)
