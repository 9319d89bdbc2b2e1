"""The fused network kernel over several tiles per workgroup: inputs and
correction operands fetched a tile ahead, ragged last tiles, both state types."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from dg_inputs import band_limited_state  # noqa: E402

pytestmark = pytest.mark.gpu


def _net(n_lon, n_lat, dtype, seed):
    import paper_2303_11767_amd as dgm
    from paper_2303_11767_amd import learned
    mesh = dgm.Mesh(n_lon, n_lat, 1, dtype=dtype, h_ref=1e4 if dtype == "f32" else 0.0)
    q, _ = band_limited_state(n_lon, n_lat, 1, 4, seed)
    q = torch.from_numpy(q).to("cuda", torch.float64 if dtype == "f64" else torch.float32)
    g = torch.Generator().manual_seed(seed)
    params = (torch.randn(learned.param_count(), generator=g) * 0.05).cuda()
    X = learned.features(mesh, q)
    fmean, fistd = X.mean(0).contiguous(), (1.0 / (X.std(0) + 1e-6)).contiguous()
    L = mesh.rhs(q).to(torch.float32).view(n_lat, n_lon, 12)
    omean = (torch.randn(n_lat, 12, generator=g).cuda() * 0.01 * L.abs().amax(1)).contiguous()
    ostd = (L.abs().amax(1) * 0.05).contiguous()
    net = learned.LearnedRHS(mesh, params, fmean, fistd, omean, ostd, kappa=1e30)
    return mesh, q, net, learned, (params, X, fmean, fistd, omean, ostd, L)


# tiles of 64 rows, 256 workgroups: less than a tile, whole tiles, a ragged
# last tile, a second tile for some workgroups (whole and ragged)
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n_lon,n_lat", [(8, 4), (16, 8), (13, 7), (128, 130), (181, 97)])
def test_corrections_of_every_row(n_lon, n_lat, dtype):
    print("[case] learned tiles", n_lon, n_lat, dtype, flush=True)
    mesh, q, net, learned, (params, X, fmean, fistd, omean, ostd, L) = _net(n_lon, n_lat, dtype, 5)
    out = net.rhs(q)
    assert net.fallbacks.item() == 0
    got = (out.double() - mesh.rhs(q).double()).view(n_lat, n_lon, 12)[:, :, 1:]
    Y = learned.mlp_forward(params, (X - fmean) * fistd).double()[:, :12].view(n_lat, n_lon, 12)
    ref = (omean.double()[:, None] + ostd.double()[:, None] * Y)[:, :, 1:]
    # the same BF16 inputs and products in both: what is left is the FP32
    # rounding of the de-standardisation (two operations on values up to twice
    # the result's parts) and, for an FP32 state, of the two right-hand sides
    bound = 2.0 ** -22 * (omean.abs().double()[:, None] + ostd.double()[:, None] * Y.abs())[:, :, 1:]
    if dtype == "f32":
        bound = bound + 2.0 ** -22 * L.abs().double()[:, :, 1:] + 2.0 ** -22 * ref.abs()
    else:
        bound = bound + 2.0 ** -40 * L.abs().double()[:, :, 1:]
    worst = ((got - ref).abs() / (bound + 1e-300)).max().item()
    print("[case]   worst of the bound", worst, flush=True)
    assert worst <= 1.0


def test_nonfinite_element_stays_in_its_stencil():
    """A non-finite element makes its 3 x 3 neighbourhood fall back and leaves
    every other element's correction as it is, those of the workgroup's later
    tiles too (what a hidden layer left in LDS is not an input)."""
    n_lon, n_lat = 181, 97
    print("[case] learned non-finite element", flush=True)
    mesh, q, net, _, _ = _net(n_lon, n_lat, "f64", 6)
    clean = net.rhs(q).view(-1, 12)
    bad = q.clone()
    e = 2 * n_lon + 40                         # a row of a first tile that has a second one
    bad.view(-1, 12)[e, 5] = float("inf")
    before = net.fallbacks.item()
    out = net.rhs(bad).view(-1, 12)
    near = {(j % n_lat) * n_lon + i for j in (1, 2, 3) for i in (39, 40, 41)}
    far = torch.tensor([k for k in range(mesh.E) if k not in near], device="cuda")
    assert net.fallbacks.item() - before == len(near)
    assert torch.equal(out[far, 1:], clean[far, 1:])
