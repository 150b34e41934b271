"""Several steps per launch on tiles (lattices below the size rule) against
single steps: the states must be bitwise identical, at the edges of the tiles'
shapes, for both precisions and models and both forms of the FP32 kick."""
import sys

import numpy as np
import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def run(xyl, spec, dtype, fusion, steps, every=0, state=None):
    lat = xyl.Lattice(spec.Lx, spec.Ly, dtype=dtype, schedule=spec.schedule, seed=spec.seed, replica=spec.replica,
                      **spec.params())
    lat.set_fusion(fusion)
    if state is None:
        lat.init_random()
    else:
        lat.set_state(*state)
    samples = []
    for n in steps:
        if every:
            samples.append(lat.step_measured(n, every))
        else:
            lat.step(n)
    out = lat.get_raw_state()
    lat.close()
    return out, samples


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("Lx,Ly,model,Jx,steps", [
    (4, 2, "xy", 1.0, [2, 3, 20]),            # the smallest lattice: one quad per row, two rows
    (8, 3, "si", -10.0, [5, 12]),             # halos that wrap onto the tile itself
    (4, 300, "xy", 1.0, [16]),                # one quad wide: whole-width tiles
    (64, 64, "xy", 0.0, [7, 30]),             # the unfactored FP32 kick
    (96, 96, "si", -10.0, [20, 1, 2]),        # short runs, each with a plan of its own
    (36, 20, "xy", -1.0, [41]),               # ferromagnetic rows
    (772, 501, "xy", 1.0, [26]),              # uneven tiles along both axes
    (1000, 7, "si", 10.0, [18]),              # few rows
    (20, 1000, "xy", 1.0, [33]),
    (512, 512, "xy", 1.0, [100]),
    (1024, 1024, "si", -10.0, [14]),          # the largest in FP64
])
def test_tiles_equal_single_steps(xyl, dtype, Lx, Ly, model, Jx, steps):
    say("tiles", dtype, Lx, Ly, model, Jx, steps)
    base = workloads.si_lattice(Lx, Ly, seed=5, replica=3) if model == "si" else \
        workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.9), (20, 0.2, 2)), seed=5, replica=3)
    base.Jx = Jx
    a, _ = run(xyl, base, dtype, 1, steps)
    b, _ = run(xyl, base, dtype, 2, steps)
    assert a[2] == b[2] == sum(steps) and a[3] == b[3]
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_tiles_between_samples_and_from_a_fresh_velocity(xyl, dtype):
    """Samples at every 1, 7 and 20 steps and a start with velocities at a late
    step: the same samples and states as single steps, bit for bit."""
    spec = workloads.LatticeSpec(128, 60, schedule=((0, 0.9), (1 << 33, 0.2)), seed=2, replica=1)
    rng = np.random.default_rng(4)
    state = (rng.uniform(-3, 3, (60, 128)).astype(np.float32), rng.normal(0, 1, (60, 128)).astype(np.float32),
             (1 << 32) - 9)
    for every in (1, 7, 20):
        a, sa = run(xyl, spec, dtype, 1, [20, 23], every, state)
        b, sb = run(xyl, spec, dtype, 2, [20, 23], every, state)
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1], b[1])
        for x, y in zip(sa, sb):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("dtype,model,sizes,budgets", [
    ("f32", "si", [(144, 144), (128, 128), (96, 80), (32, 32)], (10 ** 6, 71)),   # LDS replicas on tiles, some end
    ("f32", "xy", [(320, 40), (192, 192), (64, 64), (4, 6)], (10 ** 6, 10 ** 6)),  # a class, another width, tiny ones
    ("f32", "xy", [(1024, 512), (2048, 300), (300, 300)], (10 ** 6, 50)),          # two classes beside tiles
    ("f64", "xy", [(64, 64), (128, 60), (20, 200)], (10 ** 6, 33)),
])
def test_ensemble_tiles_equal_single_steps(xyl, dtype, model, sizes, budgets):
    """Ensembles whose replicas take several steps per launch on tiles, beside
    two-step classes, whole-in-LDS replicas and replicas that end: samples and
    states of one step per launch, bit for bit, over chunks of 25, 3 and 20
    steps, for every graph mode."""
    specs = []
    for i, (Lx, Ly) in enumerate(sizes):
        for j in range(6):
            s = workloads.si_lattice(Lx, Ly, T=1.8 + 0.05 * j, seed=j, replica=10 * i + j) if model == "si" else \
                workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.4 + 0.1 * j), (40, 0.3)), seed=j, replica=10 * i + j)
            s.nsteps = budgets[j % 2]
            if model == "xy" and j == 5:
                s.Jx = 0.0                      # the unfactored kick
            specs.append(s)
    say("ensemble tiles", dtype, model, sizes)
    res = []
    for fusion, graphs in ((1, 0), (2, 1), (2, 0), (2, 2)):
        ens = xyl.Ensemble(specs, dtype=dtype)
        ens.set_fusion(fusion)
        ens.set_graphs(graphs)
        out = [ens.step(63, every=25), ens.step(6, every=3), ens.step(80, every=20)]
        ens.step(21)
        out.append(ens.step(5, every=1000))
        res.append((out, [ens.get_state(r) for r in range(len(specs))]))
        ens.close()
    for got in res[1:]:
        for a, b in zip(res[0][0], got[0]):
            for x, y in zip(a, b):
                np.testing.assert_array_equal(x, y)
        for (ta, wa, ka), (tb, wb, kb) in zip(res[0][1], got[1]):
            assert ka == kb
            np.testing.assert_array_equal(ta, tb)
            np.testing.assert_array_equal(wa, wb)


@pytest.mark.parametrize("dtype,Lx,Ly,K,nsteps,window", [
    ("f32", 512, 300, 50, 123, 60),     # an odd window tail, a short last segment
    ("f32", 64, 64, 7, 50, 50),         # the window spans every step
    ("f32", 4, 5, 3, 10, 1),            # the smallest rows, the last state alone in the window
    ("f32", 1028, 40, 1, 6, 3),         # segments of one step (no tiles)
    ("f64", 132, 37, 25, 76, 20),       # a last segment of one step
    ("f64", 512, 64, 40, 80, 30),
])
def test_reverse_tiles_equal_single_reverse_steps(xyl, dtype, Lx, Ly, K, nsteps, window):
    """Several reverse and recompute steps per launch on tiles against single
    ones: the state adjoints bit for bit, the parameter gradients up to the
    order of their sums; and the loss window summed on tiles against the
    single steps' samples, to FP64 rounding of sums over the sites."""
    say("reverse tiles", dtype, Lx, Ly, K, nsteps, window)
    spec = dict(Jx=1.0, Jy=-0.2, h=0.4, gamma=0.8, dt=0.02, schedule=[(0, 1.1), (nsteps, 0.4)], seed=5, replica=3)
    out = []
    for fusion, adj in ((1, 1), (2, 1), (2, 2)):
        lat = xyl.Lattice(Lx, Ly, dtype=dtype, **spec)
        lat.set_fusion(fusion)
        lat.set_adjoint_fusion(adj)
        lat.init_random()
        lat.step(5)
        L = lat.adjoint_forward(nsteps, K, window)
        out.append((L,) + lat.adjoint_backward() + (lat.get_state(),))
        lat.close()
    for a in (out[0][4], out[1][4]):
        np.testing.assert_array_equal(a[0], out[2][4][0])
        np.testing.assert_array_equal(a[1], out[2][4][1])
    assert abs(out[0][0] - out[2][0]) <= 1e-12 * max(out[0][0], 1e-4)
    assert out[1][0] == out[2][0]
    np.testing.assert_array_equal(out[1][2], out[2][2])
    np.testing.assert_array_equal(out[1][3], out[2][3])
    np.testing.assert_allclose(out[2][1], out[1][1], rtol=1e-5 if dtype == "f32" else 1e-12,
                               atol=1e-9 * np.abs(out[1][1]).max())
