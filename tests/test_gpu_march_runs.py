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
