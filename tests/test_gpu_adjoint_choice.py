"""The reverse sweep takes tiles where those are faster, for the reverse steps
and for the recompute each by itself: never much slower than the sweep without
tiles (a caller's strip height selects that), and the same gradients for every
mixture of paths.

The bar of the times is 1.12: the rule leaves what measures within a few percent
undecided, and the two runs of one path differ by some 3%.  Tiles for both took
1.30 times as long at 4096 x 2048 in FP64."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def backward_us(lat, n):
    import torch
    tdt = torch.float32 if lat.dtype == 0 else torch.float64
    dth = torch.empty(lat.N, dtype=tdt, device="cuda")
    dom = torch.empty_like(dth)
    us = []
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        lat.adjoint_backward_device(dth, dom)
        e1.record()
        e1.synchronize()
        us.append(1e3 * e0.elapsed_time(e1) / n)
    return min(us[1:])


@pytest.mark.parametrize("dtype,Lx,Ly,K", [
    ("f32", 64, 64, 50), ("f32", 512, 512, 50), ("f32", 772, 501, 50), ("f32", 1024, 1024, 50), ("f32", 2048, 2048, 20),
    ("f32", 4096, 4096, 10), ("f32", 4096, 512, 20), ("f64", 64, 64, 50), ("f64", 256, 256, 50), ("f64", 512, 512, 50),
    ("f64", 1024, 1024, 20), ("f64", 1448, 1448, 20), ("f64", 2048, 1024, 20), ("f64", 2048, 2048, 20),
    ("f64", 4096, 2048, 10), ("f64", 400, 400, 50), ("f64", 560, 560, 50), ("f64", 320, 1000, 50), ("f64", 500, 2000, 20),
    ("f64", 1024, 2400, 20), ("f32", 2528, 2528, 3), ("f64", 68, 2337, 3), ("f64", 68, 2337, 50),
    ("f64", 128, 4000, 20), ("f64", 512, 512, 8),
])
def test_default_sweep_is_not_slower_than_without_tiles(xyl, dtype, Lx, Ly, K):
    import torch
    n = 4 * K
    lat = xyl.Lattice(Lx, Ly, dtype=dtype, schedule=[(0, 0.6)], seed=1,
                      stream=torch.cuda.current_stream().cuda_stream)
    lat.init_random()
    lat.adjoint_forward(n, K, K)
    us = backward_us(lat, n)
    lat.set_adjoint_fusion(2, 2)          # a caller's strips: no tiles
    untiled = backward_us(lat, n)
    say("reverse sweep", dtype, Lx, Ly, "us per step: default %.2f, without tiles %.2f" % (us, untiled))
    lat.close()
    torch.cuda.empty_cache()
    assert us <= 1.12 * untiled


@pytest.mark.parametrize("dtype,Lx,Ly,K,n", [
    ("f64", 512, 512, 20, 45),       # both on tiles
    ("f32", 4096, 4096, 5, 11),      # reverse on tiles, recompute two steps per pass, a last segment of one step
    ("f64", 2048, 2048, 6, 12),      # single reverse steps
])
def test_mixed_paths_give_the_same_gradients(xyl, dtype, Lx, Ly, K, n):
    import torch
    say("mixed reverse paths", dtype, Lx, Ly)
    out = []
    for adj in (1, 2):
        lat = xyl.Lattice(Lx, Ly, dtype=dtype, Jy=-0.2, h=0.4, schedule=[(0, 1.1), (n, 0.4)], seed=5, replica=3)
        lat.set_adjoint_fusion(adj)
        lat.init_random()
        lat.step(3)
        L = lat.adjoint_forward(n, K, 4)
        out.append((L,) + lat.adjoint_backward())
        lat.close()
        torch.cuda.empty_cache()
    assert out[0][0] == out[1][0]
    np.testing.assert_array_equal(out[0][2], out[1][2])
    np.testing.assert_array_equal(out[0][3], out[1][3])
    # sums over the sites in another order: as test_reverse_tiles_equal_single_reverse_steps
    np.testing.assert_allclose(out[1][1], out[0][1], rtol=1e-5 if dtype == "f32" else 1e-12,
                               atol=1e-9 * np.abs(out[0][1]).max())
