"""FP64 far field by expansions between well separated drops, against the
oracle's direct sums (Sec. 2.1, eq. reg_quadrature).

Tolerance: an expanded pair is truncated at 4e-15 of its potentials, and the
sums of some 1e5 terms of either side round at 1e-13 of the largest value;
1e-12 normwise per output leaves a decade."""
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


def scaled(s, radii):
    """The suspension with each drop's shape scaled about its centre."""
    off = W.drop_offsets(s.p.astype(np.int64))
    x = s.xcoef.copy()
    for d, r in enumerate(radii):
        blk = x[3 * off[d]:3 * off[d + 1]].reshape(3, -1)
        blk[:, 2:] *= r
    s.xcoef = x
    return s


def far(E, s, kinds, ntest=400):
    """(far rows, oracle's far rows at the same sampled targets, expanded pairs)."""
    import torch
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    ctx.set_drops(s.p, s.q_self, s.q_far, s.grid_mode, torch.from_numpy(s.xcoef).to(dev))
    f, sg = torch.from_numpy(s.fcoef).to(dev), torch.from_numpy(s.sigcoef).to(dev)
    u = torch.from_numpy(s.ucoef).to(dev) if s.ucoef is not None else None
    rows = E.rows_for_kinds(kinds)
    so = torch.zeros(len(rows), ctx.ntargets, dtype=torch.float64, device=dev)
    fo = torch.full_like(so, 7.0)
    ctx.layer_potentials(f, u, sg, kinds, E.FAR_FP64, so, fo)
    ctx.sync()
    direct, expanded = ctx.far_plan()
    td, tn = oracle.all_targets(s)
    sel = np.unique(np.linspace(0, len(td) - 1, ntest).astype(int))
    ref = oracle.far(s, td[sel], tn[sel])[rows]
    got = fo.cpu().numpy()[:, sel]
    ctx.close()
    return got, ref, expanded


def suspension(case):
    if case == "uneven_degrees":          # every translation class, drops of few and of many nodes
        s = W.with_separate_u(W.suspension(48, [6, 15, 29, 32], 15.0, 11))
    elif case == "uneven_sizes":          # radii from 0.2 to 1.1 about one length unit, 2p longitudes
        s = W.suspension(40, [25], 14.0, 12, grid_mode=1)
        scaled(s, np.random.default_rng(1).uniform(0.2, 1.1, 40))
    else:                                 # lowest orders only: sparse, far apart
        s = W.suspension(40, [24], 60.0, 13)
    return s


@pytest.mark.parametrize("case", ["uneven_degrees", "uneven_sizes", "sparse"])
def test_expanded_far_field_matches_the_direct_sums(E, case):
    s = suspension(case)
    got, ref, expanded = far(E, s, E.ALL_KINDS)
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)
    print(case, "expanded pairs", expanded, "err", err, flush=True)
    assert expanded > 0
    assert np.all(err < TOL), err


@pytest.mark.parametrize("away", [1e3, 1e8])
def test_suspension_far_from_the_origin(E, away):
    """Orders up to 40 and source counts that leave a rest of 2 in the moments'
    stages of four, with the whole suspension moved off the origin: the sums
    stay finite and keep the accuracy that the coordinates have there.
    Tolerance: a node's coordinates round at a few 1e-16 of `away` on either
    side, 2e-15 away together, and the kernels' relative change is at most
    six times that over the least distance, 0.2 radii; 1e-13 away, and TOL."""
    s = W.suspension(24, [32], 9.0, 17)
    ns = (s.q_far + 1) * (2 * s.q_far + 2)
    assert np.all(ns % 4 == 2)
    off = W.drop_offsets(s.p.astype(np.int64))
    for d in range(s.ndrops):
        s.xcoef[3 * off[d]:3 * off[d + 1]].reshape(3, -1)[:, 0] += np.sqrt(4.0 * np.pi) * away * np.array([1.0, -1.0, 0.5])
    got, ref, expanded = far(E, s, E.ALL_KINDS, 200)
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)
    print("away", away, "expanded pairs", expanded, "err", err, flush=True)
    assert expanded > 0
    assert np.all(err < TOL + 1e-13 * away), err


def test_truncation_of_a_distant_pair(E):
    """The double layer of two unit spheres 50 radii apart (order 10), densities
    in a bump of up to degree 48 at the points that face each other, where
    neglected orders show most (and most in this kernel), against the regular
    rule's sums in 80 bits.  Tolerance: 4e-15 of truncation (order 10 here);
    5e4 terms added in tiles of 256, sqrt(256) + sqrt(203) roundings of 1.1e-16
    for a random walk, 3.3e-15; and about ten roundings of the nodes' values,
    1e-15.  1e-14 of the vector."""
    import torch
    p, q, dist = 48, 160, 50.0
    z = np.array([0.0, 0.0, 0.5 * dist])
    s = W.two_drops(p, 1)
    nc = W.ncoef(p)
    amp = np.array([0.7, -0.4, 1.0])
    bump = [np.zeros(2 * nc) for _ in range(2)]
    for d in range(2):
        blk = s.xcoef[6 * nc * d:6 * nc * (d + 1)].reshape(3, -1)
        blk[:, 0] = np.sqrt(4.0 * np.pi) * (z if d else -z)
        for n in range(p + 1):
            e = np.sqrt((2 * n + 1) / (4.0 * np.pi)) * np.exp(-(n / 24.0) ** 2)
            bump[d][2 * W.tri(n, 0)] = e * ((-1) ** n if d else 1)
    s.fcoef = np.concatenate([a * b for b in bump for a in amp])
    s.q_self[:] = p
    s.q_far[:] = q
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    ctx.set_drops(s.p, s.q_self, s.q_far, 0, torch.from_numpy(s.xcoef).to(dev))
    assert ctx.far_plan() == (0, 2)
    so = torch.zeros(3, ctx.ntargets, dtype=torch.float64, device=dev)
    fo = torch.zeros_like(so)
    ctx.layer_potentials(None, torch.from_numpy(s.fcoef).to(dev), None, E.STOKES_DL, E.FAR_FP64, so, fo)
    ctx.sync()
    nlon = 2 * p + 2
    node = np.array([0, 5, nlon + 17, 3 * nlon + 40, 10 * nlon, 20 * nlon + 9, 40 * nlon + 60])
    got = fo.cpu().numpy()[:, node]                          # drop 0: the pole theta = 0 faces drop 1
    ctx.close()

    ld = np.longdouble
    x0, _ = oracle.targets(s, np.zeros(len(node), np.int32), node.astype(np.int32))
    x0 = x0.astype(ld) + z[:, None]
    x0 = x0 / np.sqrt((x0 ** 2).sum(0)) - z[:, None]         # on the unit sphere about -z
    ct, w = oracle.gauss_legendre(q + 1)
    ct, ph = ct.astype(ld), 2 * ld(np.pi) * np.arange(2 * q + 2).astype(ld) / (2 * q + 2)
    st = np.sqrt(1 - ct * ct)
    nrm = np.stack([np.outer(st, np.cos(ph)), np.outer(st, np.sin(ph)), np.outer(ct, np.ones_like(ph))]).reshape(3, -1)
    pn, pm, val = ct * 0 + 1, ct * 0, ct * 0                 # bump of drop 1: about the direction -z
    for n in range(p + 1):
        val = val + (2 * n + 1) / (4 * ld(np.pi)) * np.exp(-(ld(n) / 24) ** 2) * (-1) ** n * pn
        pn, pm = ((2 * n + 1) * ct * pn - n * pm) / (n + 1), pn
    dens = np.repeat(val * w.astype(ld) * 2 * ld(np.pi) / (2 * q + 2), 2 * q + 2)
    ref = np.zeros((3, len(node)), ld)
    for k in range(len(node)):
        h = x0[:, k:k + 1] - (nrm + z[:, None])
        r = np.sqrt((h * h).sum(0))
        ref[:, k] = (-6 * h * (amp.astype(ld) @ h) * (h * nrm).sum(0) / r ** 5 * dens).sum(1)
    ref /= 4 * ld(np.pi)
    err = float(np.abs(got - ref).max() / np.abs(ref).max())
    print("distant pair err", err, flush=True)
    assert err < 1e-14, err


@pytest.mark.parametrize("kinds", [1, 2, 4, 8, 16, 3, 5, 12, 18, 20, 28, 15])
def test_every_kind_set_takes_its_own_columns(E, kinds):
    got, ref, expanded = far(E, suspension("uneven_degrees"), kinds, 60)
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)
    assert expanded > 0 and np.all(err < TOL), (kinds, err)


def test_plan_follows_the_shape_and_replays(E):
    """The plan is renewed by ehd_update_shape (drops moved together: nothing
    to expand; back: the same bits), and a recorded evaluation gives them too."""
    import torch
    s = suspension("sparse")
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    x = torch.from_numpy(s.xcoef).to(dev)
    ctx.set_drops(s.p, s.q_self, s.q_far, s.grid_mode, x)
    f, sg = torch.from_numpy(s.fcoef).to(dev), torch.from_numpy(s.sigcoef).to(dev)
    out = [torch.zeros(9, ctx.ntargets, dtype=torch.float64, device=dev) for _ in range(2)]
    ctx.layer_potentials(f, None, sg, E.ALL_KINDS, E.FAR_FP64, out[0])
    ctx.sync()
    pairs = ctx.far_plan()
    assert pairs[1] > 0
    close = s.xcoef.copy().reshape(s.ndrops, 3, -1)
    close[:, :, 0] *= 0.01                # centres within a radius of each other
    ctx.update_shape(torch.from_numpy(close.ravel().copy()).to(dev))
    assert ctx.far_plan()[1] == 0
    ctx.update_shape(x)
    assert ctx.far_plan() == pairs
    for graph, overlap in ((False, False), (True, False), (True, True)):
        ctx.set_overlap(overlap)
        ctx.set_graph(graph)
        for _ in range(3):
            out[1].fill_(7.0)
            ctx.layer_potentials(f, None, sg, E.ALL_KINDS, E.FAR_FP64, out[1])
            ctx.sync()
            assert torch.equal(out[0], out[1]), (graph, overlap)
            _ = (out[1] * 2.0).sum().item()       # eager work between replays
    ctx.set_graph(False)
    ctx.close()


def lattice(nd, p, spacing=2.6):
    """nd copies of one drop on a cubic lattice."""
    one, k = W.single_drop(p=p), int(np.ceil(nd ** (1.0 / 3.0)))
    x = np.tile(one.xcoef, nd).reshape(nd, 3, -1)
    for c in range(3):
        x[:, c, 0] += np.sqrt(4.0 * np.pi) * spacing * ((np.arange(nd) // k ** c) % k)
    ps = np.full(nd, p, np.int32)
    return W.Suspension("lattice", ps, 2 * ps, 2 * ps, 0, x.ravel(), np.tile(one.fcoef, nd), np.tile(one.sigcoef, nd))


@pytest.mark.parametrize("nd, p", [(1100, 2), (1100, 8)])     # without and with expansions
def test_more_drops_than_tile_lists_are_kept_for(E, nd, p):
    s = lattice(nd, p)
    got, ref, expanded = far(E, s, E.ALL_KINDS, 60)
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)
    print(nd, p, "expanded pairs", expanded, "err", err, flush=True)
    assert (expanded > 0) == (p == 8)
    assert np.all(err < TOL), err


def test_plan_of_many_small_drops_costs_little(E):
    """No pair of drops of p = 2 is worth a translation: a new shape's time grows
    with the drops (4 times as many: 4.0 times as long without a plan), not
    with their pairs (16 times)."""
    import time
    import torch
    best = []
    for nd in (1000, 4000):
        s = lattice(nd, 2)
        ctx, x = E.Context(0), torch.from_numpy(s.xcoef).to("cuda:0")
        ctx.set_drops(s.p, s.q_self, s.q_far, 0, x)
        assert ctx.far_plan()[1] == 0
        took = []
        for _ in range(4):
            t0 = time.perf_counter()
            ctx.update_shape(x)
            took.append(time.perf_counter() - t0)
        best.append(min(took))
        ctx.close()
    print("update_shape", best, flush=True)
    assert best[1] < 6.0 * best[0], best


def test_setting_the_reported_tile_shape_changes_nothing(E):
    """ehd_set_far_config with what ehd_get_far_config reports keeps the default
    of either precision, also after another shape; another shape is followed."""
    import torch
    s = W.suspension(64, [24], 12.0, 5)                      # 80,000 targets: 7 chunks reported, 16 taken in FP64
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    ctx.set_drops(s.p, s.q_self, s.q_far, 0, torch.from_numpy(s.xcoef).to(dev))
    f = torch.from_numpy(s.fcoef).to(dev)
    shape = ctx.far_config()
    assert shape[1] < 16 and ctx.far_chunks(E.FAR_FP64) == 16 and ctx.far_chunks(E.FAR_FP32C) == shape[1]

    def run(prec):
        so = torch.zeros(3, ctx.ntargets, dtype=torch.float64, device=dev)
        fo = torch.zeros_like(so)
        ctx.layer_potentials(f, None, None, E.STOKES_SL, prec, so, fo)
        ctx.sync()
        return fo

    first = [run(k) for k in (E.FAR_FP64, E.FAR_FP32C)]
    for other in (None, (2, 3)):
        if other:
            ctx.set_far_config(*other)
            assert ctx.far_config() == other and ctx.far_chunks(E.FAR_FP64) == ctx.far_chunks(E.FAR_FP32C) == 3
            assert not torch.equal(first[1], run(E.FAR_FP32C))
        ctx.set_far_config(*shape)
        assert ctx.far_chunks(E.FAR_FP64) == 16 and ctx.far_config() == shape
        for k, want in zip((E.FAR_FP64, E.FAR_FP32C), first):
            assert torch.equal(run(k), want), (other, k)
    ctx.close()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_bad_density_stays_where_the_direct_sums_leave_it(E, bad):
    """One drop's sigma not finite: the Laplace rows of every other drop's
    targets are not finite, as by direct sums; its own targets and the Stokes
    rows are what they were."""
    import torch
    s = suspension("uneven_degrees")
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    ctx.set_drops(s.p, s.q_self, s.q_far, s.grid_mode, torch.from_numpy(s.xcoef).to(dev))
    assert ctx.far_plan()[1] > 0
    f, sg = torch.from_numpy(s.fcoef).to(dev), torch.from_numpy(s.sigcoef).to(dev)
    off, t = W.drop_offsets(s.p.astype(np.int64)), s.target_offsets()
    d = int(np.argmax(s.p))

    def run():
        so = torch.zeros(9, ctx.ntargets, dtype=torch.float64, device=dev)
        fo = torch.zeros_like(so)
        ctx.layer_potentials(f, None, sg, E.ALL_KINDS, E.FAR_FP64, so, fo)
        ctx.sync()
        return fo.cpu().numpy()

    clean = run()
    sg[off[d]] = bad
    got = run()
    ctx.close()
    own = np.zeros(clean.shape[1], bool)
    own[t[d]:t[d + 1]] = True
    assert np.array_equal(got[:6], clean[:6]) and np.array_equal(got[6:, own], clean[6:, own])
    assert not np.isfinite(got[6:, ~own]).any()


def test_plan_without_memory_sums_directly(E):
    """No room for the expansions' buffers: the same potentials by direct sums,
    and the expansions again with the next shape that finds room."""
    import torch
    s = suspension("sparse")
    ctx, dev = E.Context(0), torch.device("cuda", 0)
    close = s.xcoef.copy().reshape(s.ndrops, 3, -1)
    close[:, :, 0] *= 0.01
    x, f, sg = (torch.from_numpy(v).to(dev) for v in (s.xcoef, s.fcoef, s.sigcoef))
    ctx.set_drops(s.p, s.q_self, s.q_far, s.grid_mode, torch.from_numpy(close.ravel().copy()).to(dev))
    out = [torch.zeros(9, ctx.ntargets, dtype=torch.float64, device=dev) for _ in range(2)]
    ctx.layer_potentials(f, None, sg, E.ALL_KINDS, E.FAR_FP64, out[0])
    ctx.sync()
    assert ctx.far_plan()[1] == 0
    torch.cuda.empty_cache()
    hold = []
    for _ in range(2):
        hold.append(torch.empty(max(torch.cuda.mem_get_info()[0] - (64 << 20), 1), dtype=torch.uint8, device=dev))
    print("left", torch.cuda.mem_get_info()[0], flush=True)
    for k in range(2):
        ctx.update_shape(x)
        assert (ctx.far_plan()[1] > 0) == (k == 1)
        ctx.layer_potentials(f, None, sg, E.ALL_KINDS, E.FAR_FP64, out[k])
        ctx.sync()
        del hold[:]
        torch.cuda.empty_cache()
    ctx.close()
    err = (out[0] - out[1]).abs().max(dim=1).values / out[0].abs().max(dim=1).values
    print("err", err, flush=True)
    assert err.max().item() < TOL
