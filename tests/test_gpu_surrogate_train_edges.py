"""The training step at the edges of its branches: one row, partial and full ranges of the split gradient
reductions, more members than one optimiser launch takes, no hidden layer, layers too wide for the
fused inference; and inference right after a step, which has to see the updated weights.  Bounds: the
surrogate's for BF16 products.  The reference is the FP64 one with the operands of every product
rounded to BF16, as the step defines them: of a single row, the rounding alone (without an error of
any kernel) moves the loss by up to 0.5 %."""
import numpy as np
import pytest

from oracle import surrogate as S
from synth.surrogate import init_params, regression_data

pytestmark = pytest.mark.gpu


def bf16(a):
    import torch
    return torch.tensor(np.asarray(a, np.float64)).to(torch.bfloat16).double().numpy()


def forward(p, dims, X):
    Ws, bs = S.unflatten(np.asarray(p, np.float64), dims)
    acts, zs = [bf16(X)], []
    for W, b in zip(Ws, bs):
        zs.append(acts[-1] @ bf16(W) + b)
        acts.append(bf16(S.silu(zs[-1])))
    return zs[-1], ([bf16(W) for W in Ws], acts, zs)


def backward(cache, dY):
    Ws, acts, zs = cache
    gW, gb, dz = [None] * len(Ws), [None] * len(Ws), bf16(dY)
    for l in range(len(Ws) - 1, -1, -1):
        gW[l], gb[l] = acts[l].T @ dz, dz.sum(0)
        if l > 0:
            dz = bf16((dz @ Ws[l].T) * S.silu_grad(zs[l - 1]))
    return S.flatten(gW, gb)


@pytest.mark.parametrize("rows", [1, 63, 512, 513, 1100, 4096])
@pytest.mark.parametrize("kw, K", [(dict(din=40, width=64, depth=2, dout=3), 17), (dict(din=100, width=300, depth=1, dout=65), 2),
                                   (dict(din=70, width=1, depth=0, dout=5), 3), (dict(din=200, width=100, depth=3, dout=65), 2)])
def test_gradients_and_updated_weights(rows, kw, K):
    import torch
    from paper_1902_09171_amd import rsur
    net = rsur.Surrogate(ensemble=K, max_batch=rows, **kw)
    params = [init_params(net.dims, 21, k) for k in range(K)]
    for k, p in enumerate(params):
        net.set_params(k, p)
    X, Y = regression_data(rows, kw["din"], kw["dout"], seed=6)
    Xd, Yd = (torch.tensor(np.ascontiguousarray(a, np.float32), device="cuda:0") for a in (X, Y))
    loss = net.train_step(Xd.data_ptr(), Yd.data_ptr(), rows, 0.05)
    for k in range(K):
        Yp, cache = forward(params[k], net.dims, X)
        l_ref, dY = S.mse(Yp, Y)
        g_ref, g = backward(cache, dY), net.get_grads(k).astype(np.float64)
        # outputs within 1e-2 of their scale move the mean square by twice the mean residual
        assert abs(loss[k] - l_ref) <= 2e-2 * np.abs(Yp).max() * np.abs(Yp - Y).mean() + 1e-4 * l_ref
        assert np.linalg.norm(g - g_ref) <= 3e-2 * np.linalg.norm(g_ref), k
        nb = net.dims[-1]                              # the output layer's bias gradient, small beside the weights'
        assert np.abs((g - g_ref)[-nb:]).max() <= 3e-2 * np.abs(dY).sum(0).max(), k
    net.train_step(Xd.data_ptr(), Yd.data_ptr(), rows, 0.05, want_loss=False)
    out = torch.zeros((K, rows, kw["dout"]), device="cuda:0")
    net.forward_members(Xd.data_ptr(), rows, out.data_ptr())
    torch.cuda.synchronize()
    ref = np.stack([forward(net.get_params(k), net.dims, X)[0] for k in range(K)])
    old = np.stack([forward(p, net.dims, X)[0] for p in params])
    err = np.abs(out.cpu().numpy() - ref).max() / np.abs(ref).max()
    print(f"{kw} {rows} rows: after two steps {err:.2e}, moved {np.abs(old - ref).max() / np.abs(ref).max():.2f}", flush=True)
    assert err <= 1e-2
