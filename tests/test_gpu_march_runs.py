"""Runs on three steps per pass whose length is no multiple of six, at a size
whose last eight steps go through two-step passes (4096^2) and at a width that
those do not take (3076): the states of single steps, bit for bit, and the path."""
import sys

import numpy as np
import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("Lx,Ly,eight", [(4096, 4096, "two_step"), (3076, 2900, "march")])
def test_run_lengths(xyl, Lx, Ly, eight):
    spec = workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.9), (20, 0.2, 2)), seed=5, replica=3)
    runs = [8, 9, 20, 7]
    out = []
    for fusion in (1, 2):
        lat = xyl.Lattice(Lx, Ly, dtype="f32", schedule=spec.schedule, seed=spec.seed, replica=spec.replica,
                          **spec.params())
        lat.set_fusion(fusion)
        if fusion == 2:
            assert [lat.stepping_path(n)[0] for n in (6, 7, 8, 9, 20, 21)] == ["march"] * 2 + [eight] * 2 + ["march"] * 2
        lat.init_random()
        for n in runs:
            say("march run", Lx, Ly, "fusion", fusion, "steps", n)
            lat.step(n)
        out.append(lat.get_raw_state())
        lat.close()
    assert out[0][2] == out[1][2] == sum(runs)
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])


EDGES = [
    (4, 4), (4, 7), (8, 5), (12, 16),           # one tile that is its own neighbour, strips of four rows
    (248, 9), (252, 4), (256, 33), (260, 12),   # the widest tile, two tiles
    (496, 6), (500, 41), (1028, 300),
]


@pytest.mark.parametrize("Lx,Ly,model", [(Lx, Ly, m) for Lx, Ly in EDGES for m in ("xy", "si")] +
                         [(8192, 8192, "xy")])  # twice as many strips as run at once
def test_shapes_at_the_edges(xyl, Lx, Ly, model):
    """Shapes that the rule leaves to other paths but a tuner may give to this
    one, and the doubled strips of the largest."""
    spec = workloads.si_lattice(Lx, Ly, seed=5, replica=3) if model == "si" else \
        workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.9), (20, 0.2, 2)), seed=5, replica=3)
    runs = [7, 12] if Lx < 8192 else [7]
    say("three steps per pass", Lx, Ly, model)
    out = []
    for path in (1, 3):
        lat = xyl.Lattice(Lx, Ly, dtype="f32", schedule=spec.schedule, seed=spec.seed, replica=spec.replica,
                          **spec.params())
        assert xyl.load().xyl_choose_path(lat._h, path) == 0
        assert lat.stepping_path(12)[0] == {1: "single", 3: "march"}[path]
        lat.init_random()
        for n in runs:
            lat.step(n)
        out.append(lat.get_raw_state())
        lat.close()
    np.testing.assert_array_equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("Lx,Ly", [(3076, 2900), (4096, 4096)])
def test_samples_between_passes_are_equal(xyl, Lx, Ly):
    spec = workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.9), (20, 0.2)), seed=5, replica=3)
    out = []
    for fusion in (1, 2):
        lat = xyl.Lattice(Lx, Ly, dtype="f32", schedule=spec.schedule, seed=5, replica=3, **spec.params())
        lat.set_fusion(fusion)
        lat.init_random()
        say("sampled run", Lx, Ly, "fusion", fusion)
        out.append(lat.step_measured(25, 10))
        lat.close()
    assert out[0].shape == (3, 6)
    np.testing.assert_array_equal(out[0], out[1])
