"""The pinned places of the mass results: more contexts than a page has slots, some
freed and others made in between, each with its own result; contexts used from
two threads at once; an ensemble's members."""
import sys
import threading

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_11767_amd as dg
    return dg


def lake(mesh, h):
    q = torch.zeros(mesh.shape, dtype=mesh.dtype, device="cuda")
    q[:, 0, 0] = 2.0 * h
    return q


def test_many_contexts(dg):
    print("[case] mass of many contexts", flush=True)
    sys.stdout.flush()
    meshes = [dg.Mesh(4, 2 + k % 3, 1) for k in range(150)]
    want = [m.mass(lake(m, 1.0))[0] for m in meshes]      # the sphere's area, by the mesh
    for k in range(0, 150, 3):
        meshes[k].close()
    meshes = [dg.Mesh(4, 2 + k % 3, 1) if k % 3 == 0 else m for k, m in enumerate(meshes)]
    states = [lake(m, 1.0 + k) for k, m in enumerate(meshes)]
    torch.cuda.synchronize()
    got = {}

    def work(part):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(part, 150, 2):
                got[k] = meshes[k].mass(states[k])

    threads = [threading.Thread(target=work, args=(p,)) for p in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(150):
        assert got[k][0] == pytest.approx((1.0 + k) * want[k], rel=1e-13), k
        assert got[k][1] == 0.0 and got[k][2] == 0.0
    for m in meshes:
        m.close()


def test_members_of_an_ensemble(dg):
    print("[case] mass of ensemble members", flush=True)
    ens = dg.Ensemble([dict(n_lon=8, n_lat=4, order=k % 4) for k in range(70)], dtype="f64")
    for k, m in enumerate(ens.members):
        one = dg.Mesh(8, 4, k % 4)
        assert m.mass(lake(m, 1.0 + k))[0] == one.mass(lake(one, 1.0 + k))[0], k
        one.close()
    ens.close()
