"""Synthesis, Galerkin analysis and the surfactant solve's kernels at the edges
of their sizes (orders per block, chains per sum, blocks per dot product),
against the oracle.

Tolerance: sums of at most 5e3 terms of size one, 1e-12 normwise."""
import numpy as np
import pytest

import oracle
from paper_1811_10270_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def E():
    from paper_1811_10270_amd import ehdbim
    ehdbim.load()
    return ehdbim


def row_of_drops(E, ps, mode=0, seed=31):
    """Perturbed drops of the degrees ps, three radii apart along x."""
    import torch
    rng = np.random.default_rng(seed)
    blocks = [W._drop_shape(rng, p, (3.0 * d, 0.0, 0.0), 1.0, 0.05, 0.02)[0] for d, p in enumerate(ps)]
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    pa = np.array(ps, np.int32)
    ctx.set_drops(pa, pa, pa, mode, torch.from_numpy(np.concatenate(blocks)).to(dev))
    return ctx, dev, rng


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("ps", [[2], [3, 2], [7, 8, 9], [15, 16], [23, 24], [31, 32], [39, 40], [47, 48]])
def test_transforms_match_the_oracle(E, ps, mode):
    import torch
    ctx, dev, rng = row_of_drops(E, ps, mode)
    n, T = ctx.num_coefs(), ctx.ntargets
    for nf in (1, 3, 5):
        per = [np.concatenate([W._random_field(rng, p, 1.0, 0) for _ in range(nf)]) for p in ps]
        # buffers aligned to doubles only
        coef = torch.zeros(nf * n + 1, dtype=torch.float64, device=dev)[1:]
        coef.copy_(torch.from_numpy(np.concatenate(per)))
        grid = torch.full((nf, T), 7.0, dtype=torch.float64, device=dev)
        back = torch.full((nf * n + 1,), 7.0, dtype=torch.float64, device=dev)[1:]
        ctx.synthesize(nf, coef, grid)
        ctx.analyze(nf, grid, back)
        ctx.sync()
        got, gback = grid.cpu().numpy(), back.cpu().numpy()
        t0 = c0 = 0
        for p, c in zip(ps, per):
            nl, nlon = W.grid_dims(p, mode)
            want = oracle.synth_grid(p, c, p, mode, nf).reshape(nf, -1)
            wback = oracle.analyze_grid(p, want.ravel(), p, mode, nf).ravel()
            g, b = got[:, t0:t0 + nl * nlon], gback[c0:c0 + len(c)]
            assert np.abs(g - want).max() <= TOL * np.abs(want).max(), (p, nf)
            assert np.abs(b - wback).max() <= TOL * np.abs(wback).max(), (p, nf)
            t0 += nl * nlon
            c0 += len(c)
    ctx.close()


@pytest.mark.parametrize("ps", [[1], [4, 9], [16] * 6, [16] * 8, [32] * 4, [24] * 30, [32] * 64])
def test_surfactant_solve_leaves_no_residual(E, ps):
    """n from 6 to 71,808 unknowns: one share per dot product up to 32."""
    import torch
    ctx, dev, rng = row_of_drops(E, ps)
    n, T = ctx.num_coefs(), ctx.ntargets
    b = torch.from_numpy(np.concatenate([W._random_field(rng, p, 0.2, 0) for p in ps])).to(dev)
    kappa = rng.uniform(1e-4, 5e-2, len(ps))
    g, proj = (torch.zeros(n, dtype=torch.float64, device=dev) for _ in range(2))
    it, res = ctx.solve_surfactant(kappa, b, g, tol=1e-11)
    H, lap = (torch.zeros(T, dtype=torch.float64, device=dev) for _ in range(2))
    grad = torch.zeros(1, 3, T, dtype=torch.float64, device=dev)
    ctx.surface(H, g, grad, 1, lap)
    ctx.analyze(1, lap, proj)
    k = torch.from_numpy(np.repeat(kappa, [(p + 1) * (p + 2) for p in ps])).to(dev)
    rel = ((b - g + k * proj).norm() / b.norm()).item()
    ctx.close()
    print(len(ps), n, it, res, rel, flush=True)
    assert res <= 1e-11 and rel <= 2e-11, (it, res, rel)
