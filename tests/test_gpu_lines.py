"""Structure factor and correlation of lines with every radix of the transform
(2, 3, 4, 5, 7, 8), several lines per workgroup and part batches of them, on
both axes, against numpy's float64 transform of the same angles.

Tolerance: a transform of L points in up to ten passes leaves each Z_k within
1e-14 of the line's norm sqrt(L), so S = sum |Z|^2 / N, which is at most L, is
within 2e-14 L in the mean over the lines; 1e-13 L allows for the rotors' ulp
and the twiddle powers.  C(r) is a mean of L such terms over L.
"""
import sys

import numpy as np
import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def spectra(th, q, Jx, Jy, axis):
    Ly, Lx = th.shape
    y, x = np.mgrid[0:Ly, 0:Lx]
    s = 1 - 2 * ((x * (Jx > 0) + y * (Jy > 0)) & 1)
    z = s * np.exp(1j * q * th)
    P = np.abs(np.fft.fft(z, axis=1 - axis)) ** 2
    P = P.sum(axis=axis) / th.size
    L = len(P)
    S = 0.5 * (P + P[(-np.arange(L)) % L])
    C = np.fft.fft(S).real / L
    return S[: L // 2 + 1], C[: L // 2 + 1]


def check(lat, th, q, p):
    for axis, L in ((0, lat.Lx), (1, lat.Ly)):
        S, C = spectra(th, q, p["Jx"], p["Jy"], axis)
        np.testing.assert_allclose(lat.structure_factor(axis, L // 2), S, rtol=0, atol=1e-13 * L)
        np.testing.assert_allclose(lat.structure_factor(axis, L // 3), S[: L // 3 + 1], rtol=0, atol=1e-13 * L)
        np.testing.assert_allclose(lat.correlation(axis, L // 2), C, rtol=0, atol=1e-13)
        np.testing.assert_allclose(lat.correlation(axis, 1), C[:2], rtol=0, atol=1e-13)


@pytest.mark.parametrize("model,dtype,Lx,Ly,Jx", [
    ("xy", "f32", 4, 3, 1.0),
    ("si", "f64", 12, 5, -10.0),
    ("xy", "f64", 28, 7, -1.0),       # a radix-7 pass alone
    ("xy", "f32", 420, 21, 1.0),      # 4 3 5 7
    ("si", "f32", 360, 384, 10.0),
    ("xy", "f64", 20, 1125, 1.0),     # odd: 5 5 5 9
    ("xy", "f32", 600, 500, -1.0),
    ("xy", "f64", 3920, 6, 1.0),      # 8 2 5 7 7: radix 7 on nearly all a workgroup's points
    ("si", "f64", 4, 4096, 10.0),
    ("xy", "f32", 4096, 34, 1.0),     # 2 17: the direct sum along y
    ("xy", "f32", 3000, 2187, 1.0),   # several batches per workgroup, odd length 3^7
    ("xy", "f32", 2048, 1030, 1.0),   # 2 5 103 along y
])
def test_lines_match_float64_transform(xyl, model, dtype, Lx, Ly, Jx):
    say("lines", model, dtype, Lx, Ly, Jx)
    spec = workloads.si_lattice(Lx, Ly, Jx=Jx) if model == "si" else workloads.LatticeSpec(Lx, Ly, Jx=Jx)
    make = workloads.half_circle_state if model == "si" else workloads.random_state
    th, om = make(Lx, Ly, seed=11)
    th[: max(1, Ly // 3)] *= 0.1          # not white: part of the lines is ordered
    lat = xyl.Lattice(Lx, Ly, dtype=dtype, schedule=spec.schedule, **spec.params())
    lat.set_state(th, om)
    check(lat, lat.get_state()[0], 2.0 if model == "si" else 1.0, spec.params())
    lat.close()


def test_lines_with_angles_beyond_the_fast_reduction(xyl):
    # a caller's own buffers may hold any finite angle; what is not finite is reported
    spec = workloads.LatticeSpec(40, 24)
    th, om = workloads.random_state(40, 24, seed=3)
    lat = xyl.Lattice(40, 24, dtype="f64", schedule=spec.schedule, **spec.params())
    lat.set_state(th, om)
    th[3, 5], th[23, 39], th[7, 0], th[0, 0] = 1.0e3, -7.0e8, 64.0 + 1e-9, 63.9
    import torch
    for b in lat._bufs[:2]:
        b.copy_(torch.from_numpy(th.ravel()))
    check(lat, th, 1.0, spec.params())
    for b in lat._bufs[:2]:
        b[100] = float("nan")
    torch.cuda.synchronize()
    with pytest.raises(xyl.XylError):
        lat.structure_factor(0, 20)
    lat.close()
