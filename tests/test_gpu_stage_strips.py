"""The line layout's strips (rows of modes that are not 16-byte aligned: FP32 at
r = 1, 2, 4, 5, 6, FP64 at r = 2, 4, 6 on large meshes) at the edges of a segment:
one element, one less, exactly and one more than a wavefront holds, two segments
and a remainder; one and several rows; a forcing and every combination; nothing
written outside the state.  Bars as in the parity tests (1e-12 and 1e-5 of the
terms summed into each entry)."""
import sys

import numpy as np
import pytest

from dg_inputs import band_limited_state
from oracle import SphereDG
from parity_util import TOL, errors

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dg
    return dg


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("order", [1, 2, 4, 5, 6])
@pytest.mark.parametrize("extra", [-1, 0, 1, None])
def test_segments_f32(dg, order, extra):
    gpw = 64 // (order + 1)
    n_lon, n_lat = (1, 1) if extra is None else (2 * gpw + 1 if extra == 1 else gpw + extra, 3)
    say("strips f32", n_lon, n_lat, order)
    q, _ = band_limited_state(n_lon, n_lat, order, 3, seed=70 + order)
    m = SphereDG(n_lon, n_lat, order)
    mesh = dg.Mesh(n_lon, n_lat, order, dtype="f32", h_ref=1e4)
    mesh.kernel = "line"
    qd = torch.from_numpy(q).to("cuda", torch.float32)
    f = torch.from_numpy(np.random.default_rng(order).standard_normal(q.shape)).to("cuda", torch.float32)
    qin, fin = (t.cpu().numpy().astype(np.float64) for t in (qd, f))
    n = qd.numel()
    out = torch.full((n + 128,), 3.0, dtype=torch.float32, device="cuda")
    ref, scale = m.rhs(qin), m.rhs_scale(qin)
    for forced in (False, True):
        mesh.set_forcing(f if forced else None)
        mesh.rhs(qd, out[64:64 + n].view(mesh.shape))
        comp, _ = errors(out[64:64 + n].cpu().numpy(), ref + forced * fin, scale + forced * np.abs(fin))
        assert np.all(comp <= TOL["f32"]), (forced, comp)
        assert torch.all(out[:64] == 3.0) and torch.all(out[64 + n:] == 3.0)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("scheme", ["rk2", "rk4"])
def test_combinations(dg, scheme, dtype):
    """One step over a full and a partial segment, many layers (FP64 takes
    strips from 4096 wavefronts on): the oracle's step, every layer alike."""
    n_lon, n_lat, order, layers = 25, 3, 4, 460
    say("strips step", scheme, dtype)
    q, _ = band_limited_state(n_lon, n_lat, order, 3, seed=81)
    m = SphereDG(n_lon, n_lat, order)
    mesh = dg.Mesh(n_lon, n_lat, order, dtype=dtype, h_ref=1e4 if dtype == "f32" else 0.0)
    mesh.kernel = "line"
    mesh.levels = layers
    q1 = torch.from_numpy(q).to("cuda", mesh.dtype)
    qin = q1.cpu().numpy().astype(np.float64)
    dt, L = 20.0, m.rhs
    if scheme == "rk2":
        a = qin + dt * L(qin)
        ref = 0.5 * qin + 0.5 * (a + dt * L(a))
    else:
        k1 = L(qin)
        k2 = L(qin + 0.5 * dt * k1)
        k3 = L(qin + 0.5 * dt * k2)
        ref = qin + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + L(qin + dt * k3))
    s = {"rk2": dg.DG_SSP_RK2, "rk4": dg.DG_RK4}[scheme]
    qd = q1.expand(layers, *q1.shape).contiguous()
    mesh.rk_step(qd, mesh.empty_work(s), dt, s)
    # four stages' right-hand sides at most, weights at most 1, plus the states themselves
    scale = 4.0 * dt * m.rhs_scale(qin) + 4.0 * np.abs(qin) + 1e-3
    comp, _ = errors(qd[0].cpu().numpy(), ref, scale)
    assert np.all(comp <= TOL[dtype]), comp
    assert torch.equal(qd, qd[:1].expand_as(qd))
