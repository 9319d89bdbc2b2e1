"""The training step's row, weight-gradient and update kernels where their
partition can go wrong: one block of 32 rows, a last range shorter than the
others, ranges with fewer blocks than wavefronts, more tiles than workgroups
(over 16384 rows); inputs that are not 16-byte aligned; a mask with gaps.

Gradients against the FP64 oracle with the same BF16 rounding points, normwise
1e-3 as for the other network gradients: the sides round activations within
accumulation error of a BF16 boundary differently."""
import sys

import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("rows,shift", [(32, 1), (64, 0), (544, 3), (4128, 0), (16416, 2)])
def test_gradients_at_partition_edges(rows, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_11767_amd import learned
    say("train step", rows, shift)
    rng = np.random.default_rng(rows)
    p = mlp.init_params(rows)
    for k in ("b1", "b2", "b3"):
        p[k] = 0.1 * rng.standard_normal(p[k].shape)
    names = ("W1", "b1", "W2", "b2", "W3", "b3")
    X = rng.standard_normal((rows, 108)).astype(np.float32).astype(np.float64)
    T = rng.standard_normal((rows, 12)).astype(np.float32).astype(np.float64)
    mask = np.array([0, 1, 1, 0, 1, 1, 1, 0, 1, 1, 1, 1], dtype=np.float64)

    def off(a):      # the values `shift` floats into a buffer: aligned to 4 bytes only
        a = np.asarray(a, dtype=np.float32)
        buf = torch.zeros(a.size + shift, dtype=torch.float32, device="cuda")
        buf[shift:].copy_(torch.from_numpy(a.reshape(-1)))
        return buf[shift:].view(a.shape)

    P = off(np.concatenate([p[k].reshape(-1) for k in names]))
    n = learned.param_count()
    grads = torch.full((n + 16,), 5.0, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    learned.mlp_train_step(P, off(X), off(T), mask, grads=grads[:n], loss=loss)
    first = grads.clone()
    learned.mlp_train_step(P, off(X), off(T), mask, grads=grads[:n], loss=loss)
    assert torch.equal(first, grads)                      # fixed summation orders
    assert torch.all(grads[n:] == 5.0)
    q = {k: v.astype(np.float32).astype(np.float64) for k, v in p.items()}
    Y, cache = mlp.forward(q, X)
    g = mlp.backward(q, cache, Y, T, mask)
    ref = mlp.loss(Y, T, mask)
    assert abs(loss.item() - ref) <= 1e-4 * ref
    at = 0
    for k in names:
        got = grads[at:at + g[k].size].cpu().numpy().astype(np.float64).reshape(g[k].shape)
        at += g[k].size
        err = np.linalg.norm(got - g[k]) / np.linalg.norm(g[k])
        say("  grad", k, err)
        assert err <= 1e-3, (k, err)
