"""The FP64 r = 3 stage on the matrix cores (groups of four elements) where its
groups can go wrong: rows shorter than, equal to and just above a group, a last
group of one to three elements, one and two rows, both poles; every combination
with and without a forcing; and the numbers of groups per wavefront, which the
mesh size selects (at 3200, 24576 and 131072 groups).

The bar is the componentwise one of the parity tests, 1e-12 of the terms summed
into each entry; a step's states are compared with the same terms times dt."""
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


@pytest.mark.parametrize("n_lat", [1, 2, 5])
@pytest.mark.parametrize("n_lon", [1, 2, 3, 4, 5, 7, 8, 9])
def test_groups_at_row_ends(dg, n_lon, n_lat):
    say("m4 rhs", n_lon, n_lat)
    q, _ = band_limited_state(n_lon, n_lat, 3, 3, seed=40 + n_lon)
    m = SphereDG(n_lon, n_lat, 3)
    mesh = dg.Mesh(n_lon, n_lat, 3, dtype="f64")
    assert mesh.kernel == "half"
    out = torch.full((mesh.state_size() + 64,), 7.0, dtype=torch.float64, device="cuda")
    mesh.rhs(torch.from_numpy(q).cuda(), out[32:-32].view(mesh.shape))
    comp, _ = errors(out[32:-32].cpu().numpy(), m.rhs(q), m.rhs_scale(q))
    assert np.all(comp <= TOL["f64"]), comp
    assert torch.all(out[:32] == 7.0) and torch.all(out[-32:] == 7.0)


@pytest.mark.parametrize("forcing", [False, True])
@pytest.mark.parametrize("scheme", ["rk1", "rk2", "rk3", "rk4"])
def test_combinations(dg, scheme, forcing):
    """One step of every scheme, the stages' operands all different buffers."""
    say("m4 step", scheme, forcing)
    n_lon, n_lat = 9, 5
    q, _ = band_limited_state(n_lon, n_lat, 3, 3, seed=51)
    m = SphereDG(n_lon, n_lat, 3)
    mesh = dg.Mesh(n_lon, n_lat, 3, dtype="f64")
    dt = 50.0
    L = m.rhs
    if forcing:
        f = np.random.default_rng(5).standard_normal(q.shape)
        mesh.set_forcing(torch.from_numpy(f).cuda())
        L = lambda s: m.rhs(s) + f  # noqa: E731
    if scheme == "rk1":
        ref = q + dt * L(q)
    elif scheme == "rk2":
        q1 = q + dt * L(q)
        ref = 0.5 * q + 0.5 * (q1 + dt * L(q1))
    elif scheme == "rk3":
        q1 = q + dt * L(q)
        q2 = 0.75 * q + 0.25 * (q1 + dt * L(q1))
        ref = q / 3.0 + (2.0 / 3.0) * (q2 + dt * L(q2))
    else:
        k1 = L(q)
        k2 = L(q + 0.5 * dt * k1)
        k3 = L(q + 0.5 * dt * k2)
        ref = q + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + L(q + dt * k3))
    s = {"rk1": dg.DG_SSP_RK1, "rk2": dg.DG_SSP_RK2, "rk3": dg.DG_SSP_RK3, "rk4": dg.DG_RK4}[scheme]
    qd = torch.from_numpy(q).cuda()
    mesh.rk_step(qd, mesh.empty_work(s), dt, s)
    # four stages' right-hand sides at most, weights at most 1, plus the states themselves
    scale = 4.0 * dt * (m.rhs_scale(q) + (np.abs(f) if forcing else 0.0)) + 4.0 * np.abs(q) + 1e-3
    comp, _ = errors(qd.cpu().numpy(), ref, scale)
    assert np.all(comp <= TOL["f64"]), comp


@pytest.mark.parametrize("layers", [133, 134, 1024, 1025, 5461, 5462])
def test_groups_per_wavefront(dg, layers):
    """24 groups a layer (the last one of three elements): 3192 ..
    131088 groups, where a wavefront goes from 1 to 2, 4 and 6; every layer
    gives the bits of the single layer."""
    n_lon, n_lat = 19, 5
    say("m4 layers", layers)
    q, _ = band_limited_state(n_lon, n_lat, 3, 3, seed=60)
    mesh = dg.Mesh(n_lon, n_lat, 3, dtype="f64")
    qd = torch.from_numpy(q).cuda()
    one = mesh.rhs(qd)
    mesh.levels = layers
    got = mesh.rhs(qd.expand(layers, *qd.shape).contiguous())
    assert torch.equal(got, one.expand_as(got))
