"""FP64 r = 3 ensembles whose work items hold several groups of four elements (two,
four and six, by the groups of all members): rows shorter than an item with a
ragged last group, items across row ends cut at the member's last element, rows
of fewer than four; flat and persistent schedules, where a wavefront takes one
item after another.  Every member against its own mesh in the same layout: the
same arithmetic compiled twice, so 1e-12 of a variable's largest dq/dt (as for
the parity tests) and 1e-14 of a stage's largest value (as for other ensembles);
the values between members stay as they were."""
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# items of 8, 16 and 24 elements: over 3200, 24576 and 131072 groups
CASES = {
    8: [(7, 5), (13, 9), (3, 4), (1, 6), (5, 3), (150, 90), (8, 2), (9, 2)],
    16: [(13, 9), (7, 5), (2, 3), (450, 223), (15, 4), (17, 3), (16, 1)],
    24: [(23, 3), (13, 9), (29, 5), (5, 4), (730, 720), (24, 1), (25, 1)],
}


@pytest.mark.parametrize("item", sorted(CASES))
def test_items_of_several_groups(item):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dg
    print("[case] ensemble groups", item, flush=True)
    sys.stdout.flush()
    ens = dg.Ensemble([dict(n_lon=a, n_lat=b, order=3) for a, b in CASES[item]], dtype="f64")
    assert ens.kernel(3) == "half"
    g = torch.Generator("cuda").manual_seed(item)
    q, q0 = (torch.randn(ens.size, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    for x in (q, q0):
        for v in ens.views(x):
            v[:, 0, 0] += 2e4
    dts = [0.5 + 0.25 * k for k in range(ens.n)]
    ens.set_dt(dts)
    rhs, stage = [], []
    for m, a, b, dt in zip(ens.members, ens.views(q), ens.views(q0), dts):
        m.kernel = "half"
        rhs.append(m.rhs(a.contiguous()))
        stage.append(m.rk_stage(a.contiguous(), b.contiguous(), torch.empty_like(a), 0.75, 0.25, dt))
    for schedule in ((1, 0, 0), (4, 0, 0), (1, 256, 0), (2, 300, 0)):
        ens.set_schedule(*schedule)
        d, o = (torch.full_like(q, 7.0) for _ in range(2))
        ens.rhs(q, d)
        ens.rk_stage(q, q0, o, 0.75, 0.25)
        for k, m in enumerate(ens.members):
            dv, ov = ens.views(d)[k], ens.views(o)[k]
            for v in range(3):
                err = (dv[:, v] - rhs[k][:, v]).abs().max() / rhs[k][:, v].abs().max()
                assert err <= 1e-12, (schedule, k, v, err.item())
            err = (ov - stage[k]).abs().max() / stage[k].abs().max()
            assert err <= 1e-14, (schedule, k, err.item())
            lo, hi = ens.offsets[k] + m.state_size(), ens.offsets[k + 1]
            assert torch.all(d[lo:hi] == 7.0) and torch.all(o[lo:hi] == 7.0)
    ens.close()
