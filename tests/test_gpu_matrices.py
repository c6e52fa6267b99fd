"""Operator matrices of the solvers' mat-vecs (the singular rule of Sec. 2.1
as rows over the density's coefficients) against layer-potential evaluations,
over the degrees and grids at the edges of their tiles.

Tolerance: both sides round sums of up to 1e5 terms, 1e-13 relative; the
solves stop at a residual of 1e-12, so 1e-11 leaves a decade."""
import numpy as np
import pytest

from paper_1811_10270_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-11

# degrees, q_self of each, grid mode
CASES = [
    ([1, 2], [2, 3], 0),                 # a single term of most groups
    ([3, 8], [5, 17], 1),
    ([15, 16], [15, 33], 0),             # sixteen terms and degrees, q = p and above
    ([17, 24, 5], [34, 47, 12], 1),
    ([31, 32], [62, 65], 0),             # a seventeenth term
    ([33], [70], 1),
    ([48], [61], 0),
    ([48], [127], 0),                    # the largest rotated grid
]


@pytest.fixture(scope="module")
def E():
    from paper_1811_10270_amd import ehdbim
    ehdbim.load()
    return ehdbim


def context(E, ps, qs, mode):
    import torch
    s = W.suspension(len(ps), ps, 2.2 * len(ps) + 4.0, 21, grid_mode=mode, balanced=True)
    s.q_self[:] = [qs[ps.index(int(p))] for p in s.p]
    s.q_far[:] = np.maximum(s.p, s.q_far)
    dev = torch.device("cuda", 0)
    ctx = E.Context(0)
    ctx.set_drops(s.p, s.q_self, s.q_far, mode, torch.from_numpy(s.xcoef).to(dev))
    return s, ctx, dev


@pytest.mark.parametrize("ps, qs, mode", CASES)
def test_en_solve_matches_the_evaluating_one(E, ps, qs, mode):
    import torch
    s, ctx, dev = context(E, ps, qs, mode)
    a, b = (torch.zeros(ctx.num_coefs(), dtype=torch.float64, device=dev) for _ in range(2))
    ra = ctx.solve_En(0.4, 1.0, 0.3, a)
    rb = ctx.solve_En_noalloc(0.4, 1.0, 0.3, b)
    err = ((a - b).abs().max() / b.abs().max()).item()
    ctx.close()
    print(ps, qs, mode, "iterations", ra, rb, "err", err, flush=True)
    assert ra[1] <= 1e-12 and rb[1] <= 1e-12 and err < TOL, (ra, rb, err)


@pytest.mark.parametrize("ps, qs, mode", CASES)
def test_velocity_solve_leaves_no_residual_of_the_evaluations(E, ps, qs, mode):
    import torch
    s, ctx, dev = context(E, ps, qs, mode)
    n, T, lam = ctx.num_coefs(), ctx.ntargets, 3.0
    f = torch.from_numpy(s.fcoef).to(dev)
    u, rhs, au = (torch.zeros(3 * n, dtype=torch.float64, device=dev) for _ in range(3))
    it, res = ctx.solve_velocity(lam, f, u)
    grid = torch.zeros(3, T, dtype=torch.float64, device=dev)
    ctx.layer_potentials(f, None, None, E.STOKES_SL, E.FAR_FP64, grid)
    ctx.analyze(3, grid, rhs)
    ctx.layer_potentials(None, u, None, E.STOKES_DL, E.FAR_FP64, grid)
    ctx.analyze(3, grid, au)
    r = rhs - ((lam + 1.0) * u - (lam - 1.0) * au)
    rel = (r.norm() / rhs.norm()).item()
    ctx.close()
    print(ps, qs, mode, "iterations", it, "residual", res, "by evaluations", rel, flush=True)
    assert res <= 1e-12 and rel < TOL, (it, res, rel)


def test_solves_follow_the_shape_and_the_drops(E):
    """Matrices are built for the shapes of the solve: after ehd_update_shape
    and ehd_set_drops the solution is a fresh context's, bit for bit."""
    import torch
    s, ctx, dev = context(E, [12, 16], [24, 32], 0)

    def solve(c):
        en = torch.zeros(c.num_coefs(), dtype=torch.float64, device=dev)
        c.solve_En(0.5, 1.0, 0.0, en)
        return en

    first = solve(ctx)
    moved = s.xcoef.copy().reshape(-1)
    moved[2:] *= 1.01
    x = torch.from_numpy(moved).to(dev)
    ctx.update_shape(x)
    second = solve(ctx)
    t, other, _ = context(E, [12, 16], [24, 32], 0)
    other.update_shape(x)
    assert torch.equal(second, solve(other)) and not torch.equal(first, second)
    other.close()
    s2, ctx2, _ = context(E, [9], [18], 0)
    want = solve(ctx2)
    ctx.set_drops(s2.p, s2.q_self, s2.q_far, 0, torch.from_numpy(s2.xcoef).to(dev))
    assert torch.equal(solve(ctx), want)
    ctx.close()
    ctx2.close()


def lattice(E, nd):
    """A context of nd copies of a p = 16 drop on a cubic lattice, their force density."""
    import torch
    one, k = W.single_drop(p=16), int(np.ceil(nd ** (1.0 / 3.0)))
    x = np.tile(one.xcoef, nd).reshape(nd, 3, -1)
    for c in range(3):
        x[:, c, 0] += np.sqrt(4.0 * np.pi) * 3.0 * ((np.arange(nd) // k ** c) % k)
    ps, dev = np.full(nd, 16, np.int32), torch.device("cuda", 0)
    ctx = E.Context(0)
    ctx.set_drops(ps, 2 * ps, 2 * ps, 0, torch.from_numpy(x.ravel()).to(dev))
    return ctx, torch.from_numpy(np.tile(one.fcoef, nd)).to(dev)


def leave(nbytes):
    """Tensors that take the device's memory but for nbytes (a first one may
    free some of what the runtime holds: a second takes the rest)."""
    import torch
    torch.cuda.empty_cache()
    hold = []
    for _ in range(2):
        more = torch.cuda.mem_get_info()[0] - int(nbytes)
        if more > 1 << 21:
            hold.append(torch.empty(more, dtype=torch.uint8, device="cuda:0"))
    print("left", torch.cuda.mem_get_info()[0], "of", int(nbytes), flush=True)
    return hold


def test_solve_runs_where_matrices_and_basis_do_not_both_fit(E):
    """256 drops of p = 16: matrices 2.2 GB and 1.2 GB of weights for their build,
    basis of 200 vectors 0.38 GB.  With room for the matrices and little more
    the solve evaluates instead, as it does with next to none; large matrices
    are given back, small ones when their memory is asked for."""
    import torch
    ctx, f = lattice(E, 256)
    n, nd = ctx.num_coefs(), 256
    grid = 6 * 33 * 66 * 8
    batch = (1 << 30) // grid
    need = 48 * 578 * 306 * nd + batch * (grid + 6 * 17 * 18 * 8)
    u = [torch.zeros(3 * n, dtype=torch.float64, device="cuda:0") for _ in range(2)]
    ctx.solve_velocity(3.0, f, u[1], restart=200, maxit=4)        # (first launches take scratch memory)
    free = torch.cuda.mem_get_info()[0]
    ctx.solve_velocity(3.0, f, u[0], restart=200, tol=1e-11)
    assert abs(torch.cuda.mem_get_info()[0] - free) < 64 << 20, "matrices kept beyond the limit"
    for room in (0.15e9, -2.0e9):
        hold = leave(need + room)
        u[1].zero_()
        it, res = ctx.solve_velocity(3.0, f, u[1], restart=200, tol=1e-11)
        del hold
        err = ((u[0] - u[1]).abs().max() / u[0].abs().max()).item()
        print("room", room, "iterations", it, "residual", res, "err", err, flush=True)
        assert res <= 1e-11 and err < 1e-10
    ctx.close()
    # 64 drops: 1.8 GB kept, wanted by the next solve's larger basis (94 MB)
    ctx, f = lattice(E, 64)
    u = [torch.zeros(3 * ctx.num_coefs(), dtype=torch.float64, device="cuda:0") for _ in range(2)]
    ctx.solve_velocity(3.0, f, u[0], restart=30, tol=1e-11)
    hold = leave(80e6)
    it, res = ctx.solve_velocity(3.0, f, u[1], restart=200, tol=1e-11)
    del hold
    torch.cuda.empty_cache()
    err = ((u[0] - u[1]).abs().max() / u[0].abs().max()).item()
    ctx.close()
    assert res <= 1e-11 and err < 1e-10, (res, err)


def test_a_converged_guess_costs_one_evaluation(E):
    """A guess that meets the tolerance: its residual by one evaluation (the
    timing slots record them), no step, no matrices (1.3 GB of memory here)."""
    import torch
    s, ctx, dev = context(E, [32, 32], [64, 64], 0)
    f = torch.from_numpy(s.fcoef).to(dev)
    en = torch.zeros(ctx.num_coefs(), dtype=torch.float64, device=dev)
    u = torch.zeros(3 * ctx.num_coefs(), dtype=torch.float64, device=dev)
    ctx.solve_En(0.4, 1.0, 0.3, en)
    ctx.solve_velocity(3.0, f, u)
    ctx.close()
    _, ctx, _ = context(E, [32, 32], [64, 64], 0)
    ctx.set_timing(4)
    free = torch.cuda.mem_get_info()[0]
    for solve, v, calls in ((lambda: ctx.solve_En(0.4, 1.0, 0.3, en, tol=1e-11), en, 1),
                            (lambda: ctx.solve_velocity(3.0, f, u, tol=1e-11), u, 3)):
        want = v.clone()
        it, res = solve()
        ctx.stage_times(calls - 1)
        with pytest.raises(RuntimeError):
            ctx.stage_times(calls)
        assert it == 0 and res <= 1e-11 and torch.equal(v, want)
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20
    ctx.close()
