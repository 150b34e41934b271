"""The path that a run of steps takes, as xyl_stepping_path reports it: the
shapes that the tests of the tiles and of the three-step pass compare with
single steps do take those paths, and the settings that select a path do."""
import sys

import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def make(xyl, Lx, Ly, dtype="f32", model="xy", Jx=1.0):
    spec = workloads.si_lattice(Lx, Ly) if model == "si" else workloads.LatticeSpec(Lx, Ly)
    spec.Jx = Jx
    return xyl.Lattice(Lx, Ly, dtype=dtype, schedule=spec.schedule, **spec.params())


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("Lx,Ly,model,Jx,n", [
    (4, 2, "xy", 1.0, 20), (8, 3, "si", -10.0, 12), (4, 300, "xy", 1.0, 16), (64, 64, "xy", 0.0, 30),
    (96, 96, "si", -10.0, 20), (96, 96, "si", -10.0, 2), (36, 20, "xy", -1.0, 41), (772, 501, "xy", 1.0, 26),
    (1000, 7, "si", 10.0, 18), (20, 1000, "xy", 1.0, 33), (512, 512, "xy", 1.0, 100),
])
def test_small_lattices_take_tiles(xyl, dtype, Lx, Ly, model, Jx, n):
    lat = make(xyl, Lx, Ly, dtype, model, Jx)
    path, t = lat.stepping_path(n)
    say("path", dtype, Lx, Ly, model, n, path, t)
    assert path == "tiles" and 1 <= t <= 12
    assert lat.stepping_path(1) == ("single", 1)
    lat.set_fusion(1)
    assert lat.stepping_path(n) == ("single", 1)
    lat.close()


@pytest.mark.parametrize("Lx,Ly,model", [
    (3000, 3000, "xy"), (2564, 2503, "si"), (3076, 2900, "xy"), (8192, 1024, "xy"), (5000, 2001, "si"),
    (2052, 2052, "si"), (4096, 4096, "xy"), (4100, 4099, "xy"), (8192, 8192, "xy"),
])
def test_large_lattices_take_three_steps_per_pass(xyl, Lx, Ly, model):
    lat = make(xyl, Lx, Ly, "f32", model)
    assert lat.stepping_path(6) == ("march", 3)
    assert lat.stepping_path(500) == ("march", 3)
    assert lat.stepping_path(5)[0] == ("two_step" if lat.fusion()[1] else "single")
    if lat.fusion()[1]:
        lat.set_step2_shape(lat.fusion()[1])
        assert lat.stepping_path(500) == ("two_step", 2)
    lat.set_fusion(1)
    assert lat.stepping_path(500) == ("single", 1)
    lat.close()


def test_path_follows_the_parameters(xyl):
    # 1604^2: three steps per pass with the factored kick, tiles without it,
    # whichever the lattice had first
    for first in (1.0, 0.0):
        lat = make(xyl, 1604, 1604, Jx=first)
        for Jx in (first, 1.0 - first, first):
            lat.set_params(Jx, -0.1, 0.5, 1.0, 0.01)
            assert lat.stepping_path(60)[0] == ("march" if Jx else "tiles"), (first, Jx)
        lat.close()
