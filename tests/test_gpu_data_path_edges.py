"""Projection and stencil features at the edges of their workgroups: rows that
end inside one, fill one exactly or need several, every source order."""
import numpy as np
import pytest

from dg_inputs import band_limited_state
from oracle import SphereDG, mlp, project_order

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# a row of n_lon 3 (dst + 1) tasks against workgroups of 256
@pytest.mark.parametrize("n_lon,src,dst", [(8, 0, 0), (8, 7, 7), (86, 1, 0), (85, 4, 1), (128, 3, 1), (43, 6, 1),
                                           (43, 7, 3), (171, 2, 5), (257, 5, 0)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_projection_rows(n_lon, src, dst, dtype):
    import paper_2303_11767_amd as dgm
    from paper_2303_11767_amd import learned
    n_lat = 4
    print("[case] projection rows", n_lon, src, dst, dtype, flush=True)
    td = torch.float64 if dtype == "f64" else torch.float32
    q, _ = band_limited_state(n_lon, n_lat, src, 3, 41)
    q = torch.from_numpy(q).to("cuda", td)
    ms, md = dgm.Mesh(n_lon, n_lat, src, dtype=dtype), dgm.Mesh(n_lon, n_lat, dst, dtype=dtype)
    out = torch.full((md.E, 3, (dst + 1) ** 2), float("nan"), dtype=td, device="cuda")
    learned.project(ms, md, q, out)
    got = out.cpu().numpy().astype(np.float64)
    ref = project_order(q.cpu().numpy().astype(np.float64), SphereDG(n_lon, n_lat, src), SphereDG(n_lon, n_lat, dst))
    # FP64 sums in both types; an FP32 result is rounded once (2^-24)
    tol = 1e-12 if dtype == "f64" else 2.0 ** -23
    assert np.abs(got - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.parametrize("n_lon,n_lat", [(3, 3), (19, 7), (256, 4), (257, 5)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_features_exact(n_lon, n_lat, dtype):
    """Element order, neighbours and standardisation: the same FP32 operations, so equal bits.  The
    output starts 4 bytes past a 16-byte boundary in the second call."""
    import paper_2303_11767_amd as dgm
    from paper_2303_11767_amd import learned
    print("[case] features", n_lon, n_lat, dtype, flush=True)
    td = torch.float64 if dtype == "f64" else torch.float32
    rng = np.random.default_rng(n_lon)
    mesh = dgm.Mesh(n_lon, n_lat, 1, dtype=dtype)
    q = rng.standard_normal((mesh.E, 3, 4))
    qd = torch.from_numpy(q).to("cuda", td)
    mean = rng.standard_normal(108).astype(np.float32)
    istd = rng.standard_normal(108).astype(np.float32)
    x = mlp.stencil_features(qd.cpu().numpy(), n_lon, n_lat).astype(np.float32)
    assert np.array_equal(learned.features(mesh, qd).cpu().numpy(), x)
    out = torch.empty(mesh.E * 108 + 1, dtype=torch.float32, device="cuda")[1:].view(mesh.E, 108)
    learned.features(mesh, qd, torch.from_numpy(mean).cuda(), torch.from_numpy(istd).cuda(), out)
    assert np.array_equal(out.cpu().numpy(), (x - mean) * istd)
