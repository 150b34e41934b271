"""What an ensemble keeps between calls follows its state: samples taken without
a step after a replica's state was set, or after the launch shape was tuned, are
those of an ensemble that never had another state or shape."""
import sys

import numpy as np
import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu

SIZES = [(192, 160), (320, 96)]       # too large for the whole-in-LDS path


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def make(xyl, dtype):
    specs = [workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.7),), seed=3, replica=i) for i, (Lx, Ly) in enumerate(SIZES)]
    for s in specs:
        s.nsteps = 1 << 40
    return xyl.Ensemble(specs, dtype=dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_samples_after_a_state_was_set(xyl, dtype):
    rng = np.random.default_rng(2)
    states = [(rng.uniform(-3, 3, (Ly, Lx)).astype(np.float32), rng.normal(0, 1, (Ly, Lx)).astype(np.float32))
              for Lx, Ly in SIZES]
    want = None
    for before in (0, 10):            # the second ensemble has stepped and sampled before
        ens = make(xyl, dtype)
        if before:
            ens.step(before, every=5)
        for r, (th, om) in enumerate(states):
            ens.set_state(r, th, om, 15)
        say("samples without a step after set_state", dtype, "steps before", before)
        got = ens.step(0, every=5)
        assert [len(g) for g in got] == [1, 1]
        if want is None:
            want = got
        for a, b in zip(want, got):
            np.testing.assert_array_equal(a, b)
        # and the energy is the given state's, to FP32 rounding of its angles
        for r, (th, om) in enumerate(states):
            e_kin = 0.5 * np.mean(np.asarray(om, dtype=np.float64) ** 2)
            assert abs(got[r][0][1] - e_kin) <= 1e-5 * e_kin
        ens.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_samples_after_the_launch_shape_was_tuned(xyl, dtype):
    want = None
    for tune in (False, True):
        ens = make(xyl, dtype)
        ens.step(10)
        if tune:
            say("ensemble launch", dtype, ens.launch(), "tuned", ens.autotune())
        got = ens.step(0, every=5)
        if want is None:
            want = got
        for a, b in zip(want, got):
            np.testing.assert_array_equal(a, b)
        ens.close()
