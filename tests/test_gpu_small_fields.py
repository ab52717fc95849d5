"""The z-march on fitted tiles with fewer field points than threads (67 x 5: 483, 65 x 5: 469, 65 x 4: 402,
against 512 threads), whose last threads evaluate a point that is not kept: the evaluation, the step and the
bounds of test_gpu_fitted_tiles."""
import pytest

import test_gpu_fitted_tiles as fitted

pytestmark = pytest.mark.gpu

CASES = [((67, 67, 203), (0, 0, 0), fitted.FP64), ((129, 5, 900), (0, 1, 0), fitted.MIXED),
         ((130, 4, 1100), (1, 0, 1), fitted.MIXED), ((67, 67, 240), (1, 0, 0), fitted.NNN)]


@pytest.mark.parametrize("n,bc,kw", CASES, ids=[f"{c[0]}-{c[1]}-{i}" for i, c in enumerate(CASES)])
def test_small_fields_match_the_oracle(n, bc, kw):
    fitted.test_fitted_tiles_match_the_oracle(n, bc, kw)
