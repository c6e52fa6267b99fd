"""GPU: the perceptron kernels (forward, loss, backward, Adam) against the
FP64 numpy oracle with the same parameters, at sizes that leave ragged
64x64 tiles."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_10270_amd import ehdbim
    ehdbim.load()
    return ehdbim


@pytest.mark.parametrize("dims", [(37, 50, 3, 21, 13), (130, 96, 2, 70, 67)])
def test_forward_backward_adam_match_oracle(E, dims):
    import torch
    nin, nhid, nlay, nout, batch = dims
    dev = torch.device("cuda", 0)
    net = E.MLP(nin, nhid, nlay, nout, seed=7)
    spec, n = M.layers(nin, nhid, nlay, nout)
    assert n == net.nparams
    rng = np.random.default_rng(3)
    p = net.params().astype(np.float64)
    p[[bo + j for (_, _, b, bo) in spec for j in range(b)]] = 0.1 * rng.standard_normal(sum(b for (_, _, b, _) in spec))
    net.set_params(p.astype(np.float32))
    p = net.params().astype(np.float64)
    x = rng.standard_normal((batch, nin)).astype(np.float32)
    t = rng.standard_normal((batch, nout)).astype(np.float32)
    xd, td = torch.from_numpy(x).to(dev), torch.from_numpy(t).to(dev)
    y = torch.zeros(batch, nout, dtype=torch.float32, device=dev)
    dy = torch.zeros_like(y)
    net.forward(xd, y)
    loss = net.mse(y, td, dy)
    net.backward(dy)
    g = net.grads().astype(np.float64)
    hs = M.forward(p, spec, x.astype(np.float64))
    ref_loss, ref_dy = M.mse_and_grad(hs[-1], t.astype(np.float64))
    ref_g = M.backward(p, spec, hs, ref_dy)
    ey = np.abs(y.cpu().numpy() - hs[-1]).max() / np.abs(hs[-1]).max()
    eg = np.abs(g - ref_g).max() / np.abs(ref_g).max()
    print("mlp dims", dims, "y err", ey, "loss", loss, ref_loss, "grad err", eg, flush=True)
    assert ey < 1e-5 and abs(loss - ref_loss) < 1e-5 * ref_loss and eg < 1e-4
    net.adam(1e-3)
    p2 = net.params().astype(np.float64)
    ref_p2, _, _ = M.adam(p, g, np.zeros(n), np.zeros(n), 1, 1e-3)
    assert np.abs(p2 - ref_p2).max() < 1e-6
    net.close()


def test_training_reduces_the_loss(E):
    """Fit a random linear map: the loss falls by two orders of magnitude."""
    import torch
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(5)
    A = rng.standard_normal((32, 16)) / 6
    X = rng.standard_normal((512, 32)).astype(np.float32)
    Y = (X @ A).astype(np.float32)
    xd, yd = torch.from_numpy(X).to(dev), torch.from_numpy(Y).to(dev)
    net = E.MLP(32, 64, 2, 16, seed=11)
    out = torch.zeros(512, 16, dtype=torch.float32, device=dev)
    dy = torch.zeros_like(out)
    first = None
    for it in range(400):
        net.forward(xd, out)
        loss = net.mse(out, yd, dy, want_loss=(it % 50 == 0 or it == 399))
        if first is None:
            first = loss
        net.backward(dy)
        net.adam(3e-3)
    print("training loss", first, "->", loss, flush=True)
    assert loss < 1e-2 * first
    net.close()


@pytest.mark.parametrize("dims", [(1, 1, 1, 1, 1), (64, 128, 1, 65, 64), (63, 129, 2, 127, 65), (513, 64, 1, 3, 1),
                                  (1000, 257, 2, 191, 130), (5, 7, 1, 2, 24577)])
def test_products_at_the_edges_of_tiles_and_splits(E, dims):
    """Tiles of 64, steps of 32 and parts of at least 64 terms: sizes one below,
    at and above them, one row, sums of many parts, and more rows than one grid
    of split parts takes.  The bound is the worst-case FP32 rounding of a sum of
    K products in any order, (K + 3) units of 2^-23 of the sum of magnitudes,
    carried through the layers; an activation within its bound of zero may take
    either side of the ReLU."""
    import torch
    nin, nhid, nlay, nout, batch = dims
    dev = torch.device("cuda", 0)
    net = E.MLP(nin, nhid, nlay, nout, seed=3)
    spec, n = M.layers(nin, nhid, nlay, nout)
    rng = np.random.default_rng(8)
    p = net.params()
    p[[bo + j for (_, _, b, bo) in spec for j in range(b)]] = 0.1 * rng.standard_normal(sum(b for (_, _, b, _) in spec))
    net.set_params(p.astype(np.float32))
    p = net.params().astype(np.float64)
    x = rng.standard_normal((batch, nin)).astype(np.float32)
    gy = rng.standard_normal((batch, nout)).astype(np.float32)
    xd, gd = torch.from_numpy(x).to(dev), torch.from_numpy(gy).to(dev)
    y = torch.full((batch, nout), 7.0, dtype=torch.float32, device=dev)
    net.forward(xd, y)
    net.backward(gd)
    g = net.grads().astype(np.float64)
    u, wb = 2.0 ** -23, M.unpack(p, spec)
    hs = M.forward(p, spec, x.astype(np.float64))
    eh = [np.zeros_like(hs[0])]
    for (W, b), h in zip(wb, hs):
        eh.append(eh[-1] @ abs(W) + (len(W) + 3) * u * ((abs(h) + eh[-1]) @ abs(W) + abs(b)))
    assert (abs(y.cpu().numpy() - hs[-1]) <= eh[-1]).all()
    ref, dz, ez = M.backward(p, spec, hs, gy), gy.astype(np.float64), np.zeros(gy.shape)
    bound = np.zeros(n)
    for l in range(nlay, -1, -1):
        o, a, b, bo = spec[l]
        hm, zm = abs(hs[l]) + eh[l], abs(dz) + ez
        bound[o:o + a * b] = (hm.T @ zm * (1 + (batch + 3) * u) - abs(hs[l]).T @ abs(dz)).ravel()
        bound[bo:bo + b] = (zm * (1 + (batch + 3) * u) - abs(dz)).sum(axis=0)
        dh, W = dz @ wb[l][0].T, abs(wb[l][0]).T
        ez = ez @ W + (b + 3) * u * (zm @ W)
        ez = np.where(abs(hs[l]) <= eh[l], ez + abs(dh), np.where(hs[l] > 0, ez, 0.0))
        dz = np.where(hs[l] > 0, dh, 0.0)
    assert (abs(g - ref) <= bound + 1e-30).all()
    net.close()
