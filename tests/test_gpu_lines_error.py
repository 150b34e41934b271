"""Rounding of the structure factor's transform: no larger than that of the
direct sum that lengths other than powers of two took before they went through
it.  Against an 80-bit direct sum the direct sum in FP64 is off by 1.48e-16 (384)
and 1.54e-16 (420) of the spectrum, root mean square; the transform by 1.23e-16
and 1.02e-16 with twiddles from its table (2.30e-16 and 2.12e-16 with powers
multiplied up, which the bar, a tenth above the direct sum, refuses)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def reference(th, axis):
    Ly, Lx = th.shape
    x = np.mgrid[0:Ly, 0:Lx][1]
    s = (1 - 2 * (x & 1)).astype(np.longdouble)          # Jx > 0 > Jy
    t = th.astype(np.longdouble)
    c, n = s * np.cos(t), s * np.sin(t)
    if axis == 1:
        c, n = c.T, n.T
    L = c.shape[1]
    m = np.arange(L)
    a = np.longdouble("6.28318530717958647692528676655900577") * m / L
    idx = np.outer(m, m) % L
    W, V = np.cos(a)[idx], np.sin(a)[idx]
    re, im = c @ W + n @ V, n @ W - c @ V
    P = (re * re + im * im).sum(axis=0) / th.size
    return ((P + P[(-m) % L]) / 2)[: L // 2 + 1]


@pytest.mark.parametrize("Lx,Ly,axis", [(384, 360, 0), (384, 360, 1), (420, 300, 0)])
def test_transform_rounds_no_worse_than_the_direct_sum(xyl, Lx, Ly, axis):
    assert np.finfo(np.longdouble).eps < 1e-18
    lat = xyl.Lattice(Lx, Ly, dtype="f32", schedule=[(0, 1.5), (600, 0.0)], seed=7)
    lat.init_random()
    lat.step(300)
    L = (Lx, Ly)[axis]
    S, R = lat.structure_factor(axis, L // 2), reference(lat.get_state()[0], axis)
    err = float(np.sqrt(np.mean((S - R) ** 2) / np.mean(R * R)))
    print("structure factor", Lx, Ly, axis, "rms error %.2e" % err, file=sys.stderr, flush=True)
    lat.close()
    assert err <= 1.1 * 1.54e-16


@pytest.mark.parametrize("axis", [0, 1])
def test_correlation_adds_no_rounding_of_its_sum(xyl, axis):
    """C(r) from the spectrum: within half an ulp of C(0) = 1 (1.1e-16) of an
    80-bit pair sum, where a plain sum of the spectrum was off by 1.7e-16 and
    2.2e-16 (the pair sums in FP64 by 2e-17)."""
    lat = xyl.Lattice(384, 360, dtype="f32", schedule=[(0, 1.5), (600, 0.0)], seed=7)
    lat.init_random()
    lat.step(300)
    th = lat.get_state()[0].astype(np.longdouble)
    x = np.mgrid[0:360, 0:384][1]
    s = (1 - 2 * (x & 1)).astype(np.longdouble)
    c, n = s * np.cos(th), s * np.sin(th)
    L = (384, 360)[axis]
    want = np.array([(c * np.roll(c, -r, axis=1 - axis) + n * np.roll(n, -r, axis=1 - axis)).sum() / th.size
                     for r in range(L // 2 + 1)])
    err = float(np.abs(lat.correlation(axis, L // 2) - want).max())
    print("correlation", axis, "max error %.2e" % err, file=sys.stderr, flush=True)
    lat.close()
    assert err <= 1.15e-16
