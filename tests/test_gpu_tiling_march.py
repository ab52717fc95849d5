"""The check of test_gpu_tiling.py, bit for bit between the 64 x 8 and the 64 x 4 build, for the z-march:
grids of up to 2^19 nodes take bricks, which have no tile, unless a chunk length is asked for, and many
larger ones take fitted tiles.  Here the small cases march in chunks of 1, 3 and 7 planes (64 x 8 against
64 x 4 tiles, line-tied and periodic, concave maps), and four larger grids take what the library chooses:
128 x 90 x 48 and 64 x 129 x 70 64-wide tiles with rows to spare in both builds, 129 x 70 x 70 tiles of
65 x 7 against 65 x 3, 70 x 110 x 75 of 35 x 14 against 35 x 7."""
import pytest

import paper_1405_0942_amd as R
import test_gpu_tiling as tiling

pytestmark = pytest.mark.gpu

SMALL = ("concave_70x11x37_pxy", "concave_20x18x16_lt", "twist_16_lt_adaptive")
LARGE = [((128, 90, 48), (0, 0, 0), {}), ((64, 129, 70), (1, 1, 1), {}), ((129, 70, 70), (0, 1, 0), {}),
         ((70, 110, 75), (1, 0, 0), dict(precision=R.RELAX_FP32_MIXED))]


@pytest.mark.parametrize("tz", [1, 3, 7])
@pytest.mark.parametrize("name", SMALL)
def test_march_independent_of_tile_height(name, tz, monkeypatch):
    monkeypatch.setenv("RELAX_TZ", str(tz))
    tiling.test_results_independent_of_tile_height(name)


@pytest.mark.parametrize("n,bc,kw", LARGE, ids=[str(c[0]) for c in LARGE])
def test_chosen_tiles_independent_of_tile_height(n, bc, kw, monkeypatch):
    name = f"{n}-{bc}"
    case = (lambda: tiling._concave_case(n, bc, 0.7, 4.0), dict(dt0=1e-4, adaptive=False, **kw), 3)
    monkeypatch.setitem(tiling.CASES, name, case)
    tiling.test_results_independent_of_tile_height(name)
