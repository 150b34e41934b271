"""The loss window of a long run between few checkpoints is summed in pieces of
bounded scratch on tiles: one million window steps take no gigabyte of partial
sums, and the loss is that of a run whose checkpoints cut the window into
other pieces."""
import sys

import pytest

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def test_window_scratch_is_bounded(xyl):
    import torch
    Lx, Ly, W = 128, 128, 600_000
    used, loss = [], []
    for K in (W, 10_000):
        lat = xyl.Lattice(Lx, Ly, dtype="f32", schedule=[(0, 0.9)], seed=3)
        lat.init_random()
        assert lat.stepping_path(min(K, W))[0] == "tiles"
        lat.step(64)
        lat.sync()
        free0 = torch.cuda.mem_get_info()[0]
        say("window", W, "checkpoints every", K)
        loss.append(lat.adjoint_forward(W, K, W))
        used.append(free0 - torch.cuda.mem_get_info()[0])
        lat.close()
    say("scratch of the window of %d steps: %.0f MB" % (W, used[0] / 1e6), "losses", loss)
    # 48 bytes a step for the samples and their sums, 64 MB of partial sums
    assert used[0] <= 48 * W + (64 << 20) + (64 << 20)
    assert loss[0] == loss[1]
