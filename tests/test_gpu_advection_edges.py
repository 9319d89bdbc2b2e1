"""Linear advection at the edges of its partition: meshes of one row or column
(an element is its own neighbour), fewer elements than a wavefront's four, a last
workgroup that is not full, both kernels (the FP64 r = 3 one on the matrix cores
and the general one), and every scheme's combinations.  Bars as in the other
advection tests: 1e-12 (FP64) and 2e-5 (FP32) of the largest value."""
import sys

import numpy as np
import pytest

from oracle.advection import AdvectionDG

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


@pytest.mark.parametrize("order,dtype", [(3, "f64"), (3, "f32"), (2, "f64"), (5, "f64")])
@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 5), (3, 1), (2, 2), (4, 4), (5, 7), (17, 1), (16, 9)])
def test_rhs_small_meshes(dg, nx, ny, order, dtype):
    say("advection edges", nx, ny, order, dtype)
    m = AdvectionDG(nx, ny, order, lx=1.3, ly=0.7, beta=(0.6, -1.1))
    q = np.random.default_rng(nx * 100 + ny).standard_normal((nx * ny, m.N))
    td = torch.float64 if dtype == "f64" else torch.float32
    adv = dg.Advection(nx, ny, order, lx=1.3, ly=0.7, beta=(0.6, -1.1), dtype=dtype)
    qd = torch.from_numpy(q).to("cuda", td)
    ref = m.rhs(qd.cpu().numpy().astype(np.float64))
    n = qd.numel()
    out = torch.full((n + 128,), 9.0, dtype=td, device="cuda")
    adv.rhs(qd, out[64:64 + n].view(qd.shape))
    err = np.abs(out[64:64 + n].cpu().numpy().reshape(ref.shape) - ref).max() / np.abs(ref).max()
    say("  max relative", err)
    assert err <= (1e-12 if dtype == "f64" else 2e-5)
    assert torch.all(out[:64] == 9.0) and torch.all(out[64 + n:] == 9.0)


@pytest.mark.parametrize("order,dtype", [(3, "f64"), (2, "f32")])
@pytest.mark.parametrize("scheme", ["rk1", "rk2", "rk3", "rk4"])
def test_step_of_every_scheme(dg, scheme, order, dtype):
    say("advection step", scheme, order, dtype)
    nx, ny = 6, 5
    m = AdvectionDG(nx, ny, order, beta=(-0.8, 1.0))
    q = np.random.default_rng(3).standard_normal((nx * ny, m.N))
    td = torch.float64 if dtype == "f64" else torch.float32
    adv = dg.Advection(nx, ny, order, beta=(-0.8, 1.0), dtype=dtype)
    qd = torch.from_numpy(q).to("cuda", td)
    q = qd.cpu().numpy().astype(np.float64)
    dt, L = 1e-3, m.rhs
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
    adv.rk_step(qd, adv.empty_work(s), dt, s)
    err = np.abs(qd.cpu().numpy() - ref).max() / np.abs(ref).max()
    say("  max relative", err)
    assert err <= (1e-12 if dtype == "f64" else 2e-5)
