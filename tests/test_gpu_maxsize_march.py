"""Three steps per pass on lattices just under 2^31 sites (4229 column tiles of
rows of 2^20 sites, and 187 of a square one) against single steps: every angle
and velocity bit for bit, noise and the periodic seam included, over one pair of
passes and the single step that is left."""
import sys

import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("Lx,Ly", [(46336, 46336), (1 << 20, 2046)])
def test_largest_lattices_three_steps_per_pass(xyl, Lx, Ly):
    import torch
    n = 7
    say("max size, three steps per pass", Lx, Ly)
    spec = workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.9), (20, 0.2)), seed=9, replica=5)
    lat = xyl.Lattice(Lx, Ly, dtype="f32", schedule=spec.schedule, seed=9, replica=5, **spec.params())
    try:
        assert lat.stepping_path(n) == ("march", 3)
        lat.init_random()
        lat.step(n)
        theta, u = lat.theta_tensor().clone(), lat._bufs[2].clone()
        lat.init_random()
        lat.set_fusion(1)
        lat.step(n)
        lat.sync()
        assert torch.equal(lat.theta_tensor(), theta)
        assert torch.equal(lat._bufs[2], u)
    finally:
        lat.close()
        torch.cuda.empty_cache()
