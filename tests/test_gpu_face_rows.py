"""The accuracy of the one-sided rows on line-tied faces: u of the sweeps against the same formulas in 80 bits,
on boxes whose faces lie at powers of two (+-1, +-4), where a node just outside the box has half the accuracy of
those inside.

The bound: no further from the 80-bit u, rms, than the plain FP64 evaluation of the one-sided rows is (which the
fused products of the sweeps undercut by a tenth), with a tenth for other roundings.  Rows taken as central
differences with a ghost node outside the box are 1.4 times as far."""
import numpy as np
import pytest

import workloads as W
from gpu_util import banner, context, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _difference(v, axis, ends):
    """v(+e) - v(-e) along x (0), y or z; with `ends` the one-sided rows on the faces, else 0 there."""
    v = np.moveaxis(v, 3 - axis, 0)
    d = np.zeros_like(v)
    d[1:-1] = v[2:] - v[:-2]
    if ends:
        d[0] = (4 * v[1] - 3 * v[0]) - v[2]
        d[-1] = v[-3] - (4 * v[-2] - 3 * v[-1])
    return np.moveaxis(d, 0, 3 - axis)


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _cross(a, b):
    return np.stack([a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]])


def _velocity(x, B0, h, kind):
    """u = J x B, all faces line-tied, in the number type `kind`."""
    x, h = x.astype(kind), [kind(v) for v in h]
    q = [4 * h[1] * h[2] * B0[0].astype(kind), 4 * h[2] * h[0] * B0[1].astype(kind), 4 * h[0] * h[1] * B0[2].astype(kind)]
    F = [_difference(x, a, True) for a in range(3)]
    D = _dot(F[0], _cross(F[1], F[2]))
    B = (F[0] * q[0] + F[1] * q[1] + F[2] * q[2]) / D
    G = [_difference(B, a, False) for a in range(3)]
    c = [_dot(F[(k + 2) % 3], G[(k + 1) % 3]) - _dot(F[(k + 1) % 3], G[(k + 2) % 3]) for k in range(3)]
    u = _cross((F[0] * c[0] + F[1] * c[1] + F[2] * c[2]) / D, B)
    for a in range(1, 4):
        np.moveaxis(u, a, 0)[[0, -1]] = 0
    return u


@pytest.mark.parametrize("tz", [None, 9], ids=["chosen", "march"])
@pytest.mark.parametrize("n,half", [((51, 51, 51), (4.0, 4.0, 10.0)), ((70, 40, 33), (4.0, 1.0, 1.0)), ((129, 70, 70), (4.0, 4.0, 4.0))])
def test_rows_on_faces_are_as_accurate_as_inside(n, half, tz, monkeypatch):
    if tz is not None:
        monkeypatch.setenv("RELAX_TZ", str(tz))
    g = W.make_grid(n, [(-v, v) for v in half], (0, 0, 0))
    z, y, x = np.meshgrid(*[np.linspace(-half[a], half[a], n[a]) for a in (2, 1, 0)], indexing="ij")
    wall = np.prod([np.cos(0.5 * np.pi * v / w) for v, w in zip((x, y, z), half)], axis=0)
    X = np.stack([x, y, z]) + 0.05 * min(half) * wall * np.stack([np.sin(y + z), np.cos(x - z), np.sin(x + y)])
    twist = 0.4 * z * np.exp(-(x ** 2 + y ** 2) / 2 - z ** 2 / 4)
    B0 = np.stack([y * twist, -x * twist, np.ones_like(x)])
    banner(f"face rows {n} {half} chunk {tz}")
    with context(g, X, B0, dt0=1e-4, adaptive=False) as r:
        u = host(r.velocity())
    ref = _velocity(X, B0, g.h, np.longdouble)
    rms = [float(np.sqrt(np.mean((v - ref) ** 2))) for v in (u, _velocity(X, B0, g.h, np.float64))]
    print(f"rms error of u: {rms[0]:.3e}, plain FP64 {rms[1]:.3e}, ratio {rms[0] / rms[1]:.3f}")
    assert rms[0] <= 1.1 * rms[1]
