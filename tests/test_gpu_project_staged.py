"""The projection's staged form (source rows through LDS: FP32 onto up to half of a
row's values, FP64 onto a fifth) at the edges of a workgroup of 256 tasks: rows of
one element, that fill one exactly, that leave a task for the next one, and whose
elements straddle two (three values a row do not divide 256).

Sums are FP64 in both types, an FP32 result is rounded once (2^-24)."""
import numpy as np
import pytest

from dg_inputs import band_limited_state
from oracle import SphereDG, project_order

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,src,dst", [("f32", s, d) for s in range(1, 8) for d in range((s + 1) // 2)] +
                         [("f64", s, 0) for s in range(4, 8)])
@pytest.mark.parametrize("n_lon", [1, 85, 86, 128, 171])
def test_staged_projection(n_lon, dtype, src, dst):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dgm
    from paper_2303_11767_amd import learned
    n_lat = 3
    print("[case] staged projection", n_lon, src, dst, dtype, flush=True)
    td = torch.float64 if dtype == "f64" else torch.float32
    q, _ = band_limited_state(n_lon, n_lat, src, 3, 43)
    q = torch.from_numpy(q).to("cuda", td)
    ms, md = dgm.Mesh(n_lon, n_lat, src, dtype=dtype), dgm.Mesh(n_lon, n_lat, dst, dtype=dtype)
    n = md.E * 3 * (dst + 1) ** 2
    buf = torch.full((n + 128,), 3.0, dtype=td, device="cuda")
    learned.project(ms, md, q, buf[64:64 + n].view(md.shape))
    assert torch.all(buf[:64] == 3.0) and torch.all(buf[64 + n:] == 3.0)
    got = buf[64:64 + n].cpu().numpy().astype(np.float64).reshape(md.shape)
    ref = project_order(q.cpu().numpy().astype(np.float64), SphereDG(n_lon, n_lat, src), SphereDG(n_lon, n_lat, dst))
    tol = 1e-12 if dtype == "f64" else 2.0 ** -23
    assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
