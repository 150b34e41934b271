"""Domain labelling at the edges of its tiles (32 x 32 sites): part tiles, tiles
that wrap onto themselves, single rows, spins of every density, lines and
checkerboards; labels, sizes and counts equal the oracle's exactly, in repeated
calls too (each clears what the one before left; large label arrays take
another way to the host from the second call on)."""
import sys

import numpy as np
import pytest

import oracle
from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def spins(kind, Lx, Ly, rng):
    y, x = np.mgrid[0:Ly, 0:Lx]
    if kind == "checker":
        return (x + y) % 2
    if kind == "columns":
        return (x // 3) % 2
    if kind == "comb":                       # a row of teeth: long chains within and across tiles
        return ((x % 2 == 0) | (y % 37 == 0)).astype(int)
    return (rng.random((Ly, Lx)) < float(kind)).astype(int)


@pytest.mark.parametrize("dtype,Lx,Ly", [
    ("f32", 4, 2), ("f64", 32, 32), ("f32", 36, 31), ("f32", 64, 33), ("f64", 28, 70),
    ("f32", 100, 5), ("f32", 1028, 600),
])
def test_domains_equal_oracle(xyl, dtype, Lx, Ly):
    spec = workloads.LatticeSpec(Lx, Ly, seed=1)
    o = oracle.Oracle(**spec.oracle_kwargs())
    lat = xyl.Lattice(Lx, Ly, dtype=dtype, schedule=spec.schedule, seed=1, **spec.params())
    rng = np.random.default_rng(9)
    for kind in ("0.5", "0.59", "0.05", "1.0", "checker", "columns", "comb"):
        say("domains", dtype, Lx, Ly, kind)
        th = np.where(spins(kind, Lx, Ly, rng) > 0, 0.25, -3.0)
        lat.set_state(th, np.zeros_like(th))
        lab_o, nd_o = o.domains(th, 32 if dtype == "f32" else 64)
        sz = np.bincount(np.unique(lab_o, return_inverse=True)[1].ravel())
        want_s, want_c = np.unique(sz, return_counts=True)
        for labels, sizes, counts, nd, mx in (lat.domains(), lat.domains(want_labels=False), lat.domains()):
            assert nd == nd_o and mx == want_s[-1]
            np.testing.assert_array_equal(sizes, want_s)
            np.testing.assert_array_equal(counts, want_c)
            if labels is not None:
                np.testing.assert_array_equal(labels, lab_o)
    lat.close()
