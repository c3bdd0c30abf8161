"""surrogate.train and surrogate.predict hand device buffers to a context whose stream torch does not know: a
minibatch must stay as it is until the step that reads it has run, and nothing may be left to write into a
result.  On the CPU with every enqueued step put off until the program waits, the worst that a device may do; on
the GPU against a loop that waits after every step, bit for bit."""
import ctypes
import types

import numpy as np
import pytest


def problem(n, din, dout, seed=4):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((n, din)), rng.standard_normal((n, dout))


class LateNet:
    """Stands in for a context: train_step is enqueued, and its batch is read when the device is waited for."""

    def __init__(self, din, dout, max_batch):
        self.din, self.dout, self.max_batch, self.pending, self.seen = din, dout, max_batch, [], []

    def fit_norm(self, *a):
        pass

    def train_step(self, x, y, b, lr, want_loss=True):
        self.pending.append((x, y, b))
        if want_loss:
            self.wait()
            return np.zeros(1, np.float32)

    def wait(self):
        for x, y, b in self.pending:
            rows = lambda p, d: np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_float)), (b, d)).copy()
            self.seen.append((rows(x, self.din), rows(y, self.dout)))
        self.pending = []


@pytest.mark.parametrize("log_every", [0, 3])
def test_a_step_reads_its_own_minibatch(log_every):
    import torch
    from paper_1902_09171_amd import surrogate as SU
    X, Y = problem(40, 5, 2)
    net = LateNet(5, 2, 8)
    late = types.SimpleNamespace(**{k: getattr(torch, k) for k in ("float32", "index_select")},
                                 tensor=lambda a, **k: torch.tensor(a), empty=lambda s, dtype, device: torch.empty(s, dtype=dtype),
                                 Generator=lambda device: torch.Generator(),
                                 randperm=lambda n, generator, device: torch.randperm(n, generator=generator),
                                 cuda=types.SimpleNamespace(synchronize=net.wait))
    SU.train(late, net, X, Y, steps=12, batch=8, seed=7, log_every=log_every)
    gen, want = torch.Generator().manual_seed(7), []
    for t in range(12):
        if t % 5 == 0:
            perm = torch.randperm(40, generator=gen)
        want.append(perm[(t % 5) * 8:(t % 5 + 1) * 8].numpy())
    assert len(net.seen) == 12
    for (x, y), idx in zip(net.seen, want):
        assert np.array_equal(x, X[idx].astype(np.float32)) and np.array_equal(y, Y[idx].astype(np.float32))


@pytest.mark.gpu
def test_training_equals_a_loop_that_waits():
    import torch
    from paper_1902_09171_amd import rsur, surrogate as SU
    from synth.surrogate import init_params
    X, Y = problem(20000, 153, 6)
    out = []
    for wait in (False, True, False):
        net = rsur.Surrogate(din=153, width=256, depth=4, dout=6, ensemble=5, max_batch=4096)
        for k in range(5):
            net.set_params(k, init_params(net.dims, 31, k))
        if wait:
            step = net.train_step

            def train_step(*a, **k):
                r = step(*a, **k)
                torch.cuda.synchronize()
                return r
            net.train_step = train_step
        SU.train(torch, net, X, Y, steps=100, batch=2048, lr=2e-3, lr_final=2e-4, seed=3)
        out.append([net.get_params(k) for k in range(5)] + list(SU.predict(torch, net, X[:300])))
        net.close()
    for o in (out[0], out[2]):
        assert all(np.array_equal(a, b) for a, b in zip(o, out[1]))
