"""GPU: the singular self-interaction at the edges of its column schedule
(groups of four Legendre columns, zero to three columns left over), of its
rotation jobs and of its row tiles (one to five, cos/sin terms in registers,
reloaded, in LDS and from memory), every field set, against the FP64 oracle.

Tolerance: both sides round sums of up to 1e5 terms, 1e-13 relative; 1e-10 as
for the other FP64 parity tests."""
import numpy as np
import pytest

import oracle
from paper_1811_10270_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-10

CASES = [(1, 2, 0), (2, 3, 1), (3, 7, 0), (4, 4, 1), (7, 20, 0), (9, 18, 1), (11, 127, 0), (14, 28, 0), (16, 127, 0),
         (17, 34, 0), (19, 40, 1), (22, 44, 0), (24, 127, 0), (24, 126, 1), (25, 50, 0), (27, 54, 1), (30, 60, 0),
         (32, 127, 0), (33, 66, 0), (35, 50, 1), (37, 75, 0), (40, 80, 0), (46, 92, 0), (46, 127, 0), (47, 94, 1),
         (48, 48, 0), (48, 127, 1)]


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_10270_amd import ehdbim
    ehdbim.load()
    return ehdbim


@pytest.mark.parametrize("p, q, mode", CASES)
def test_self_interaction_at_schedule_edges(E, p, q, mode):
    import torch
    s = W.suspension(1, [p], 6.0, 100 + p, grid_mode=mode)
    s.q_self[:] = q
    s.q_far[:] = np.maximum(s.p, s.q_far)
    dev = torch.device("cuda", 0)
    ctx = E.Context(0)
    ctx.set_drops(s.p, s.q_self, s.q_far, mode, torch.from_numpy(s.xcoef).to(dev))
    f, sg = torch.from_numpy(s.fcoef).to(dev), torch.from_numpy(s.sigcoef).to(dev)
    td, tn = oracle.all_targets(s)
    sel = np.unique(np.random.default_rng(p).integers(0, len(td), 24))
    ref = oracle.self_(s, td[sel], tn[sel])
    worst = 0.0
    for a, u, b, kinds in ((f, None, sg, E.ALL_KINDS), (f, None, None, E.STOKES_SL | E.STOKES_DL), (None, f, None, E.STOKES_DL),
                           (None, None, sg, E.LAP_SL | E.LAP_DL | E.LAP_DLADJ)):
        rows = E.rows_for_kinds(kinds)
        out = torch.zeros(len(rows), ctx.ntargets, dtype=torch.float64, device=dev)
        ctx.layer_potentials(a, u, b, kinds, E.FAR_FP64, out)
        ctx.sync()
        want = ref[rows]
        err = np.abs(out.cpu().numpy()[:, sel] - want).max(axis=1) / np.abs(want).max(axis=1)
        worst = max(worst, err.max())
    ctx.close()
    print("self", p, q, mode, "err", worst, flush=True)
    assert worst < TOL
