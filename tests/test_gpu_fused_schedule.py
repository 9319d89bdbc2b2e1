"""The single fused launch is open, without setting layouts first, to ensembles of
members that are large enough for the line layout each by itself (over 512
wavefronts of it at r >= 4, 2048 below), and its right-hand sides are those of the
per-order launches to rounding (the parity bars, of a variable's largest value)."""
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,members", [
    ("f32", [(120, 60, 5)]),                    # 720 wavefronts of the line layout
    ("f32", [(100, 60, 5), (111, 54, 5)]),      # 600 and 648
    ("f32", [(180, 89, 5), (73, 74, 6)]),       # 1602 and 666
    ("f32", [(90, 45, 7)]),                     # 540
    ("f32", [(265, 130, 3), (360, 180, 2)]),    # 2210 and 3240
    ("f64", [(112, 55, 4), (265, 115, 2)]),     # 550 and 1495: line by the order's total
])
def test_fused_launch_of_large_members(dtype, members):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dg
    print("[case] fused schedule", dtype, members, flush=True)
    sys.stdout.flush()
    ens = dg.Ensemble([dict(n_lon=a, n_lat=b, order=r) for a, b, r in members], dtype=dtype,
                      h_ref=1e4 if dtype == "f32" else 0.0)
    assert all(ens.kernel(r) == "line" for _, _, r in members)
    g = torch.Generator("cuda").manual_seed(9)
    q = torch.randn(ens.size, dtype=ens.dtype, device="cuda", generator=g)
    for v in ens.views(q):
        v[:, 0, 0] += 2e4
    outs = []
    for fused in (False, True):
        ens.set_schedule(1, 0, fused)
        assert ens.schedule()[2] is fused
        outs.append(ens.rhs(q))
    for a, b in zip(*(ens.views(o) for o in outs)):
        for v in range(3):
            err = (a[:, v] - b[:, v]).abs().max() / a[:, v].abs().max()
            assert err <= (1e-12 if dtype == "f64" else 1e-5), (v, err.item())
    ens.close()
