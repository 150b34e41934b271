"""xyl_set_step2_shape selects the two-step pass where the lattice can take it,
changes nothing elsewhere, and holds until xyl_autotune."""
import pytest

from paper_2409_06412_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Lx,Ly,shaped", [
    ("f32", 512, 512, "two_step"),
    ("f32", 4096, 2048, "two_step"),
    ("f32", 772, 501, "tiles"),       # a width that the two-step pass does not take
    ("f32", 2052, 2052, "march"),
    ("f64", 512, 64, "tiles"),
])
def test_shape_holds_where_it_applies(xyl, dtype, Lx, Ly, shaped):
    spec = workloads.LatticeSpec(Lx, Ly, schedule=((0, 0.6),), seed=1)
    lat = xyl.Lattice(Lx, Ly, dtype=dtype, schedule=spec.schedule, seed=1, **spec.params())
    lat.init_random()
    before = lat.stepping_path(60)
    lat.set_step2_shape(8)
    assert lat.stepping_path(60)[0] == shaped
    if shaped != "two_step":
        assert lat.stepping_path(60) == before
    lat.set_step2_shape()             # (0 keeps the values)
    assert lat.stepping_path(60)[0] == shaped
    if Lx == 512 and dtype == "f32":
        # tiles 1.3 us per step, two steps per pass 3.0
        lat.autotune()
        assert lat.stepping_path(60) == before
    lat.close()
