"""The fused inference kernel at the edges of its tiles: one row to several blocks of either row count,
narrow, wide and absent hidden layers, more outputs than one feature tile, and pre-activations so
negative that e^-z overflows.  Bounds: the surrogate's for BF16 products against the FP64 reference."""
import numpy as np
import pytest

from oracle import surrogate as S
from synth.surrogate import init_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 31, 33, 127, 129, 4097])
@pytest.mark.parametrize("kw, K", [(dict(din=153, width=256, depth=4, dout=6), 5), (dict(din=9, width=64, depth=1, dout=33), 2),
                                   (dict(din=70, width=130, depth=2, dout=64), 3), (dict(din=20, width=1, depth=0, dout=5), 1)])
def test_members_against_the_reference(rows, kw, K):
    import torch
    from paper_1902_09171_amd import rsur
    net = rsur.Surrogate(ensemble=K, max_batch=rows, **kw)
    params = [init_params(net.dims, 3, k) for k in range(K)]
    for k, p in enumerate(params):
        net.set_params(k, p)
    rng = np.random.default_rng(rows)
    X = rng.standard_normal((rows, kw["din"])).astype(np.float32)
    Xd = torch.tensor(X, device="cuda:0")
    out = torch.full((K, rows + 1, kw["dout"]), 7.0, device="cuda:0")
    net.forward_members(Xd.data_ptr(), rows, out.data_ptr())
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(-1)
    n = K * rows * kw["dout"]
    assert np.all(got[n:] == 7.0)                      # nothing past the last row
    ref = np.stack([S.forward(p, net.dims, X)[0] for p in params])
    assert np.abs(got[:n].reshape(ref.shape) - ref).max() <= 1e-2 * np.abs(ref).max()


@pytest.mark.parametrize("rows", [40, 5000])
def test_very_negative_activations(rows):
    import torch
    from paper_1902_09171_amd import rsur
    kw = dict(din=64, width=64, depth=2, dout=4)
    net = rsur.Surrogate(ensemble=5, max_batch=rows, **kw)
    rng = np.random.default_rng(1)
    params = []
    for k in range(5):
        p = init_params(net.dims, 8, k)
        p[:64 * 64] *= 60.0                            # z of either sign up to a few hundred: e^-z overflows
        params.append(p)
        net.set_params(k, p)
    X = rng.standard_normal((rows, 64)).astype(np.float32)
    mean = torch.zeros((rows, 4), device="cuda:0")
    net.forward(torch.tensor(X, device="cuda:0").data_ptr(), rows, mean.data_ptr(), None)
    torch.cuda.synchronize()
    Ws, bs = S.unflatten(params[0], net.dims)
    assert (X @ Ws[0] + bs[0]).min() < -100.0
    ref = np.mean([S.forward(p, net.dims, X)[0] for p in params], 0)
    got = mean.cpu().numpy()
    assert np.all(np.isfinite(got)) and np.abs(got - ref).max() <= 1e-2 * np.abs(ref).max()
