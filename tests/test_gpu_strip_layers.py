"""Line layout on both sides of the launch's switch from rows to strips (taken
where a launch, all layers together, has enough wavefronts): a layer among many
has the same bits as the same state alone, at every order whose rows are not
16-byte aligned, with a full and a partial last segment, with and without a
forcing, for the right-hand side and for every combination of states."""
import sys

import pytest

from dg_inputs import band_limited_state, random_plane_state

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("forced", [False, True])
@pytest.mark.parametrize("plane", [False, True])
@pytest.mark.parametrize("dtype,order", [("f64", r) for r in (0, 2, 4, 6)] + [("f32", r) for r in (0, 1, 2, 4, 5, 6)])
def test_layer_among_many_equals_the_layer_alone(dtype, order, plane, forced):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dg
    print("[case] strip layers", dtype, order, plane, forced, flush=True)
    sys.stdout.flush()
    n_lon, n_lat = 2 * (64 // (order + 1)) + 1, 3      # three wavefronts a row, the last one element
    many = 456                                         # 4104 wavefronts
    href = (1e4 if not plane else 1e3) if dtype == "f32" else 0.0
    if plane:
        mesh = dg.Plane(n_lon, n_lat, order, 4e5, 1e5, dtype=dtype, h_ref=href)
        q = random_plane_state(n_lon, n_lat, order, 4e5, 1e5, 7)
    else:
        mesh = dg.Mesh(n_lon, n_lat, order, dtype=dtype, h_ref=href)
        q, _ = band_limited_state(n_lon, n_lat, order, 3, seed=7)
    mesh.kernel = "line"
    q = torch.from_numpy(q).to("cuda", mesh.dtype).view(mesh.shape)
    f = torch.randn(q.shape, dtype=mesh.dtype, device="cuda", generator=torch.Generator("cuda").manual_seed(order))

    def run(layers, what):
        mesh.levels = layers
        shape = mesh.shape
        x = q.expand(shape).contiguous() if layers > 1 else q.clone()
        mesh.set_forcing((f.expand(shape).contiguous() if layers > 1 else f) if forced else None)
        x = mesh.rhs(x) if what == "rhs" else mesh.rk_step(x, mesh.empty_work(what), 0.5, what, 2)
        mesh.set_forcing(None)
        mesh.levels = 1
        return x

    for what in ("rhs", dg.DG_SSP_RK2, dg.DG_SSP_RK3, dg.DG_RK4):
        one, all_ = run(1, what), run(many, what)
        assert torch.isfinite(one).all()
        assert torch.equal(all_, one.expand_as(all_)), what
