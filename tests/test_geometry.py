"""The choice of tiles and chunks (relax.cpp) as relax_workspace_bytes shows it, on the CPU."""
import math
import time
import types

import pytest

import paper_1405_0942_amd as R


def _config(n, **kw):
    g = types.SimpleNamespace(n=n, h=(0.1, 0.1, 0.1), bc=(R.RELAX_PERIODIC,) * 3)
    return R.make_config(g, dt0=1e-3, **kw)


@pytest.mark.parametrize("n", [(4, 2 ** 26 - 1, 4096), (4, 2 ** 25, 4096), (4, 2 ** 24, 2 ** 14), (8, 2 ** 25 - 1, 2048)])
def test_workspace_of_the_widest_grids_holds_the_partial_records(n):
    """Twelve FP64 vectors, and for each 64 x 8 tile of the x-y plane at least one record of eight doubles
    and one Lambda: also where tiles times chunks pass 2^32."""
    tiles = -(-n[0] // 64) * -(-n[1] // 8)
    assert R.relax_workspace_bytes(_config(n)) >= 12 * 24 * n[0] * n[1] * n[2] + tiles * 72


@pytest.mark.parametrize("n", [(16384, 16383, 4), (4, 4, 2 ** 22)])
def test_choosing_the_geometry_of_wide_and_long_grids_takes_little_time(n):
    """Every call without a context chooses its geometry: some 60 tile widths and 2 sqrt(nz) chunk lengths
    are a few ten microseconds, a walk over all tile heights or chunk counts took 10 ms."""
    cfg, best = _config(n), math.inf
    for _ in range(7):
        t = time.perf_counter()
        assert R.relax_workspace_bytes(cfg) > 0
        best = min(best, time.perf_counter() - t)
    assert best < 2e-3


def test_a_recorded_step_keeps_what_the_reverse_sweeps_read():
    """A longer checkpoint segment holds, for each step more, x_n, k_1 and y_3 to y_6: six FP64 vectors (and
    no other checkpoint, with one slot for K_record = 4 steps either way)."""
    n = (32, 32, 32)
    a, b = (R.relax_workspace_bytes(_config(n, record=True, checkpoint_every=c), 4) for c in (5, 9))
    assert b - a == 4 * 6 * 24 * n[0] * n[1] * n[2]
