"""What an ensemble keeps between calls follows its state: samples taken without
a step after a replica's state was set, or after the launch shape was tuned, are
those of an ensemble that never had another state or shape; and the plan follows each
chunk's length, whichever length came first."""
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


def mixed(xyl, dtype, model, budgets=(1 << 40,)):
    sizes = [(64, 64), (96, 96), (128, 128), (144, 144), (320, 40), (192, 192)] if dtype == "f32" else \
        [(64, 64), (128, 60), (20, 200)]
    specs = []
    for i, (Lx, Ly) in enumerate(sizes):
        for j in range(8):
            s = workloads.si_lattice(Lx, Ly, T=1.8 + 0.02 * j, seed=j, replica=10 * i + j) if model == "si" else \
                workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.4 + 0.1 * j), (40, 0.3)), seed=j, replica=10 * i + j)
            s.nsteps = budgets[(i + j) % len(budgets)]
            specs.append(s)
    return xyl.Ensemble(specs, dtype=dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_the_first_chunk_decides_nothing_for_later_ones(xyl, dtype):
    want = {}
    for first in (0, 1, 2, 5, 200):
        ens = mixed(xyl, dtype, "si")
        if first:
            ens.step(first)
            if first < 4:
                assert "tiles" not in ens.paths() and "two_step" not in ens.paths()
        for n in (200, 12, 5):
            ens.step(n)
            got = ens.paths()
            assert want.setdefault(n, got) == got, (first, n)
        assert "tiles" in want[200]
        ens.close()
    say("ensemble paths", dtype, want[200])


@pytest.mark.parametrize("graphs", [0, 1, 2])
@pytest.mark.parametrize("dtype,model", [("f32", "xy"), ("f32", "si"), ("f64", "xy")])
def test_chunks_of_every_length_equal_single_steps(xyl, dtype, model, graphs):
    """Chunks of one to two hundred steps in turn, with and without samples, and
    replicas that end in between: the samples and states of single steps, bit
    for bit."""
    say("chunk lengths", dtype, model, graphs)
    res = []
    for fusion in (1, 2):
        ens = mixed(xyl, dtype, model, budgets=(1 << 40, 97, 1 << 40, 240, 110))
        ens.set_fusion(fusion)
        ens.set_graphs(graphs)
        out = []
        for n, every in ((2, 0), (60, 20), (3, 1), (5, 5), (30, 6), (1, 0), (12, 0), (24, 12), (40, 2), (8, 0), (90, 30),
                         (7, 0), (60, 20), (60, 20)):
            got = ens.step(n, every=every)
            if every:
                out.append(got)
        out.append(ens.step(0, every=1))
        res.append((out, [ens.get_state(r) for r in range(ens.n)]))
        ens.close()
    for a, b in zip(res[0][0], res[1][0]):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
    for (ta, wa, ka), (tb, wb, kb) in zip(res[0][1], res[1][1]):
        assert ka == kb
        np.testing.assert_array_equal(ta, tb)
        np.testing.assert_array_equal(wa, wb)
