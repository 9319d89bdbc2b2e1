"""Default layouts of an ensemble's orders: by the size of all members of an
order together, whatever the members' own sizes."""
import pytest

from dg_inputs import band_limited_state

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# r = 2: at most 1024 wavefronts of the line layout half, more line (a 42x22
# FP32 member has 2 x 22, a 63x16 one 3 x 16)
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("count,want", [(1, "half"), (23, "half"), (24, "line")])
def test_layout_of_many_small_members(dtype, count, want):
    import paper_2303_11767_amd as dgm
    print("[case] ensemble default layouts", dtype, count, flush=True)
    members = [dict(n_lon=42, n_lat=22, order=2) for _ in range(count)] + [dict(n_lon=20, n_lat=10, order=4)]
    ens = dgm.Ensemble(members, dtype=dtype, h_ref=1e4 if dtype == "f32" else 0.0)
    assert ens.kernel(2) == want and ens.kernel(4) == "half"
    q = ens.empty_state()
    dts = []
    for k, (m, v) in enumerate(zip(ens.members, ens.views(q))):
        qh, info = band_limited_state(m.n_lon, m.n_lat, m.order, 4, 70 + k)
        v.copy_(torch.from_numpy(qh).to(v.dtype))
        dts.append(dgm.cfl_time_step(m, info.cmax, 0.1))
    ens.set_dt(dts)
    out = ens.empty_state()
    ens.rk_stage(q, None, out, 0.0, 1.0)
    for k in (0, count - 1, count):
        m, qv = ens.members[k], ens.views(q)[k]
        m.kernel = ens.kernel(m.order)
        ref = torch.empty_like(qv)
        m.rk_stage(qv.contiguous(), None, ref, 0.0, 1.0, dts[k])
        err = (ens.views(out)[k].double() - ref.double()).abs().max().item() / ref.double().abs().max().item()
        # the same arithmetic, compiled twice: multiply-adds may differ
        assert err <= (1e-14 if dtype == "f64" else 1e-6), (k, err)
