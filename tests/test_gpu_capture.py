"""Steps issued while the caller captures the lattice's stream, and steps of a
lattice whose second velocity buffer does not fit: nothing is allocated and no
graph of the library's is launched inside a capture, and either way the run
falls to single steps with the same states, bit for bit.  For every path of long
runs, in runs shorter and longer than the library's own graphs (32 steps)."""
import ctypes
import sys

import numpy as np
import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu

SHAPES = [
    ("f32", 512, 96, "tiles"),
    ("f64", 64, 48, "tiles"),
    ("f32", 2564, 2503, "march"),
    ("f32", 4096, 1024, "two_step"),      # shaped: the two-step pass by itself
    ("f32", 2052, 2052, "single"),        # fusion 1
]


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def make(xyl, dtype, Lx, Ly, path, stream=None):
    spec = workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.9), (100, 0.2)), seed=5, replica=3)
    lat = xyl.Lattice(Lx, Ly, dtype=dtype, schedule=spec.schedule, seed=5, replica=3, stream=stream, **spec.params())
    if path == "two_step":
        lat.set_step2_shape(8)
    if path == "single":
        lat.set_fusion(1)
    lat.init_random()
    assert lat.stepping_path(12)[0] == path
    return lat


def reference(xyl, dtype, Lx, Ly, runs):
    lat = make(xyl, dtype, Lx, Ly, "single")
    out = []
    for n in runs:
        lat.step(n)
        out.append(lat.get_raw_state())
    lat.close()
    return out


def same(a, b):
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


@pytest.mark.parametrize("n", [8, 40])
@pytest.mark.parametrize("dtype,Lx,Ly,path", SHAPES)
def test_steps_inside_a_capture(xyl, dtype, Lx, Ly, path, n):
    import torch
    want = reference(xyl, dtype, Lx, Ly, [n, n])
    s = torch.cuda.Stream()
    for first in (True, False):
        # the lattice's first step (no second velocity buffer yet), or one after
        # an eager run has made it
        say("capture", dtype, Lx, Ly, path, "steps", n, "first call" if first else "after a run")
        lat = make(xyl, dtype, Lx, Ly, path, stream=s.cuda_stream)
        if not first:
            lat.step(n)
        start = lat.get_raw_state()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            lat.step(n)
        assert lat.step_index == start[2] + n
        for rep in range(3):
            # (an even run ends in the buffer that its start lies in)
            lat.set_raw_state(start[0], start[1], start[2], start[3])
            lat.sync()
            torch.ones(1000, device="cuda").sum().item()
            g.replay()
            torch.cuda.synchronize()
            same(lat.get_raw_state(), want[0 if first else 1])
        # and eager steps go on from there
        lat.set_raw_state(start[0], start[1], start[2], start[3])
        lat.step(n)
        same(lat.get_raw_state(), want[0 if first else 1])
        lat.close()


@pytest.mark.parametrize("n", [8, 41])
@pytest.mark.parametrize("dtype,Lx,Ly,path", SHAPES)
def test_steps_without_a_second_buffer(xyl, dtype, Lx, Ly, path, n):
    say("no second buffer", dtype, Lx, Ly, path, n)
    want = reference(xyl, dtype, Lx, Ly, [n])[0]
    lat = make(xyl, dtype, Lx, Ly, path)
    assert xyl.load().xyl_deny_second_buffer(lat._h) == 0
    assert lat.stepping_path(n) == ("single", 1)
    lat.step(n)
    same(lat.get_raw_state(), want)
    assert xyl.load().xyl_deny_second_buffer(ctypes.c_void_p()) == -1
    lat.close()
