"""The network calls' scratch belongs to one call: calls in flight on two streams,
of growing sizes, never get the same memory, and training steps interleaved on
two streams, and run from two threads, give the bits of the same steps one after
the other."""
import sys
import threading

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MASK = [0] + [1] * 11


@pytest.fixture(scope="module")
def learned():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_11767_amd import learned
    return learned


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


class Net:
    """One network's state and batches of growing size."""

    def __init__(self, learned, seed):
        g = torch.Generator("cuda").manual_seed(seed)

        def rnd(*shape):
            return torch.randn(*shape, device="cuda", generator=g)
        self.learned = learned
        self.p = 0.05 * rnd(learned.param_count())
        self.m, self.v = torch.zeros_like(self.p), torch.zeros_like(self.p)
        self.grads, self.loss = torch.zeros_like(self.p), torch.zeros(1, device="cuda")
        self.batches = [(rnd(n, 108), rnd(n, 12)) for n in (96, 2048, 96, 4096, 8192, 2048)]
        self.losses = []

    def step(self, k, stream=None):
        X, T = self.batches[k]
        self.learned.mlp_train_step(self.p, X, T, MASK, self.m, self.v, k + 1, 1e-3, self.grads, self.loss,
                                    stream=stream)

    def result(self):
        return torch.cat([self.p, self.m, self.v, self.grads, self.loss])


def serial(learned, seed):
    net = Net(learned, seed)
    for k in range(len(net.batches)):
        net.step(k)
    torch.cuda.synchronize()
    return net.result()


def test_steps_on_two_streams(learned):
    say("training steps on two streams")
    ref = [serial(learned, s) for s in (1, 2)]
    nets = [Net(learned, s) for s in (1, 2)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in range(len(nets[0].batches)):
        for net, s in zip(nets, streams):
            net.step(k, s)
    torch.cuda.synchronize()
    for net, r in zip(nets, ref):
        assert torch.equal(net.result(), r)


def test_steps_from_two_threads(learned):
    say("training steps from two threads")
    ref = [serial(learned, s) for s in (3, 4)]
    nets = [Net(learned, s) for s in (3, 4)]
    torch.cuda.synchronize()

    def work(net):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(len(net.batches)):
                net.step(k)
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(n,)) for n in nets]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for net, r in zip(nets, ref):
        assert torch.equal(net.result(), r)


def test_scratch_of_calls_in_flight_is_disjoint(learned, monkeypatch):
    say("scratch of calls in flight")
    lib, seen = learned.load(), []
    real = {name: getattr(lib, name) for name in ("dg_mlp_forward", "dg_mlp_train_step")}

    class Recorder:
        def __getattr__(self, name):
            if name not in real:
                return getattr(lib, name)

            def call(*args):
                seen.append(args[-2].value)            # workspace, stream
                return real[name](*args)
            return call

    monkeypatch.setattr(learned, "load", lambda: Recorder())
    nets = [Net(learned, s) for s in (5, 6)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k in (0, 1):                                   # the second one needs a larger scratch
        X = nets[0].batches[k][0]
        outs = [torch.empty(X.shape[0], 12, device="cuda") for _ in streams]
        torch.cuda.synchronize()
        del seen[:]
        for net, s, o in zip(nets, streams, outs):
            net.step(k, s)
            learned.mlp_forward(net.p, X, o, stream=s)
        b = learned.ctypes.c_int64()
        assert lib.dg_mlp_workspace_size(X.shape[0], learned.ctypes.byref(b)) == 0
        first, second = seen[:2], seen[2:]             # by stream
        assert len(first) == len(second) == 2
        assert all(abs(x - y) >= b.value for x in first for y in second)
        torch.cuda.synchronize()
