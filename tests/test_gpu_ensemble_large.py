"""FP32 line items of ensembles on both sides of the flat kernels' switch (three
packed states against the 256 MiB Infinity Cache): orders 2 and 5, which take rows
below it and strips above, members with partial last segments and of one element,
each against its own mesh (the same arithmetic compiled more than once: 1e-6 of a
stage's largest value, 1e-5 of a variable's largest dq/dt); the values between
members stay as they were."""
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SMALL = [(1, 1), (21, 3), (22, 2), (101, 50), (10, 4), (9, 3)]


@pytest.mark.parametrize("order", [2, 5])
@pytest.mark.parametrize("large", [False, True])
def test_rows_and_strips(order, large):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dg
    print("[case] ensemble large", order, large, flush=True)
    sys.stdout.flush()
    n = {2: 14, 5: 4}[order] if large else 1               # 907200 and 259200 elements of the large ones
    ens = dg.Ensemble([dict(n_lon=a, n_lat=b, order=order) for a, b in SMALL + [(360, 180)] * n], dtype="f32", h_ref=1e4)
    ens.set_kernel(order, "line")
    assert (3 * 4 * ens.size > 256 << 20) is large
    g = torch.Generator("cuda").manual_seed(order)
    q, q0 = (torch.randn(ens.size, dtype=torch.float32, device="cuda", generator=g) for _ in range(2))
    for x in (q, q0):
        for v in ens.views(x):
            v[:, 0, 0] += 2e4
    dts = [0.5 + 0.25 * k for k in range(ens.n)]
    ens.set_dt(dts)
    for schedule in ((1, 0, 0), (2, 0, 0)):
        ens.set_schedule(*schedule)
        d, o = (torch.full_like(q, 7.0) for _ in range(2))
        ens.rhs(q, d)
        ens.rk_stage(q, q0, o, 0.75, 0.25)
        for k in list(range(len(SMALL))) + [ens.n - 1]:
            m = ens.members[k]
            m.kernel = "line"
            a, b = (ens.views(x)[k].contiguous() for x in (q, q0))
            rhs, stage = m.rhs(a), m.rk_stage(a, b, torch.empty_like(a), 0.75, 0.25, dts[k])
            dv, ov = ens.views(d)[k], ens.views(o)[k]
            for v in range(3):
                assert (dv[:, v] - rhs[:, v]).abs().max() <= 1e-5 * rhs[:, v].abs().max(), (schedule, k, v)
            assert (ov - stage).abs().max() <= 1e-6 * stage.abs().max(), (schedule, k)
            lo, hi = ens.offsets[k] + m.state_size(), ens.offsets[k + 1]
            assert torch.all(d[lo:hi] == 7.0) and torch.all(o[lo:hi] == 7.0)
    ens.close()
