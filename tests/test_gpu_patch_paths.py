"""The 25-31-point patch kernels and the 17-21-point two-row kernels at the edges of
what they accept, against the FP64 CPU oracle at sampled nodes: no atoms, as many
atom images as a region can hold, short and long recurrences, recurrences that end
early, non-finite potentials, bounds that are too tight, and batches that mix cube
sides.  Every case says which kernels it is for.

Tolerances as in the other parity tests: bounds 1e-12 of the largest |eigenvalue|,
FP64 moments 1e-10; mixed moments 1e-5 (n_pl 12: twelve FP32 roundings of up to
2^-24, each carried at most 6-fold and doubled by the product formulas, are 8.6e-6).
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1708_07913_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07913_amd import sq
    sq.load_library()
    torch.cuda.set_device(0)


def assert_kernels(g, cube, chains):
    """The launch group of the context: cube side, projector chains, default shape."""
    from paper_1708_07913_amd import sq
    assert sq.Batch([g], [1.0]).groups() == [(cube, chains, 0)]


def compare(g, o, nodes, moments=True):
    lo, hi = (t.cpu().numpy() for t in g.spectral_bounds())
    lo_ref, hi_ref = o.bounds(nodes=nodes)
    scale = max(np.abs(lo_ref).max(), np.abs(hi_ref).max())
    assert np.abs(lo[nodes] - lo_ref).max() < 1e-12 * scale
    assert np.abs(hi[nodes] - hi_ref).max() < 1e-12 * scale
    if moments:
        m = g.moments().cpu().numpy()
        assert np.isfinite(m).all()
        assert np.abs(m[nodes] - o.moments(lo[nodes], hi[nodes], nodes=nodes)).max() < 1e-10


def sample(g, count=4):
    return np.unique(np.r_[0, g.nd - 1, np.random.default_rng(1).choice(g.nd, count, replace=False)])


def on_grid(natom, n, h, npl=12, seed=2):
    """natom atoms on grid points of an n^3 mesh, each sphere that one point: a cube of
    n points holds exactly natom images, whatever its node."""
    at = np.random.default_rng(seed).choice(n ** 3, natom, replace=False)
    xyz = np.stack([at % n, at // n % n, at // n ** 2], 1) * h
    kb = np.tile([0.7, 0.5 * h, 0.5], (natom, 1))
    V = -1.0 + np.random.default_rng(seed + 1).random(n ** 3)
    return xyz, kb, V


@pytest.mark.parametrize("cube", [25, 27, 29, 31])
@pytest.mark.parametrize("natom", [0, 1, 255, 256])
def test_number_of_images(cube, natom):
    from paper_1708_07913_amd import sq
    print(f"case {cube} points, {natom} images", flush=True)
    h = 0.4
    args = (cube * h, h, 12, (cube // 2) * h, 12, 0.04)
    xyz, kb, V = on_grid(natom, cube, h)
    g = sq.SQ(*args, xyz, kb, torch.from_numpy(V).cuda())
    assert_kernels(g, cube, 1)
    o = oracle.Oracle(*args, xyz, kb, V)
    nodes = sample(g, 2)
    if natom:
        assert all(o.region_images(int(q)) == natom for q in nodes)
    compare(g, o, nodes)


def test_more_images_than_slots_is_an_error():
    from paper_1708_07913_amd import sq
    h, cube = 0.4, 25
    xyz, kb, V = on_grid(257, cube, h)
    g = sq.SQ(cube * h, h, 12, 12 * h, 12, 0.04, xyz, kb, torch.from_numpy(V).cuda())
    assert_kernels(g, cube, 1)
    with pytest.raises(sq.SQError):
        g.spectral_bounds()


@pytest.mark.parametrize("cell,cube,steps", [((1, 8.0, 0.5, 2.5), 11, 256), ((1, 9.0, 0.55, 4.4), 17, 256),
                                             ((1, 8.0, 0.5, 5.0), 21, 200), ((1, 7.78, 0.5, 6.5), 27, 1),
                                             ((1, 7.78, 0.5, 6.5), 27, 2), ((1, 7.78, 0.5, 6.5), 27, 256)])
def test_lengths_of_the_recurrence(cell, cube, steps):
    """The extremes have converged long before 200 steps; 1 and 2 are their own values."""
    from paper_1708_07913_amd import sq
    print(f"case {cube} points, {steps} steps", flush=True)
    cells, a, h, rcut = cell
    wl = W.fcc_workload(f"c{cube}", cells, a, 0.1, 5, h, rcut, 12, 1.0)
    V = wl.veff()
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda(), n_lanczos=steps)
    assert_kernels(g, cube, 1)
    compare(g, oracle.Oracle.from_workload(wl, veff=V, n_lanczos=steps), sample(g, 2), moments=steps > 2)


@pytest.mark.parametrize("cube", [25, 29])
def test_recurrence_that_ends_early(cube):
    """beta_0 below 1e-13 of the diagonal: one step, lmin = lmax = alpha_0."""
    from paper_1708_07913_amd import sq
    h, n = 0.5, 16
    args = (n * h, h, 12, (cube // 2) * h, 12, 0.04)
    V = np.full(n ** 3, 1e16)
    g = sq.SQ(*args, [], [], torch.from_numpy(V).cuda())
    assert_kernels(g, cube, 1)
    nodes = sample(g)
    lo, hi = (t.cpu().numpy() for t in g.spectral_bounds())
    assert np.array_equal(lo, hi)
    lo_ref, hi_ref = oracle.Oracle(*args, np.zeros((0, 3)), np.zeros((0, 3)), V).bounds(nodes=nodes)
    assert np.array_equal(lo_ref, hi_ref)
    assert np.abs(lo[nodes] - lo_ref).max() < 1e-12 * 1e16


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_non_finite_potential_is_an_error(bad):
    from paper_1708_07913_amd import sq
    wl = W.fcc_workload("c29", 1, 7.78, 0.1, 5, 0.5, 7.0, 12, 1.0)
    V = wl.veff()
    V[77] = bad
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda())
    assert_kernels(g, 29, 1)
    with pytest.raises(sq.SQError):
        g.spectral_bounds()


@pytest.mark.parametrize("cube,h,rcut", [(25, 0.5, 6.0), (31, 0.4, 6.0)])
def test_bounds_that_are_too_tight_are_an_error(cube, h, rcut):
    from paper_1708_07913_amd import sq
    wl = W.fcc_workload("tight", 1, 7.78, 0.1, 5, h, rcut, 32, 1.0)
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(wl.veff()).cuda())
    assert_kernels(g, cube, 1)
    lo, hi = g.spectral_bounds()
    mid = 0.5 * (lo + hi)
    g.set_bounds(mid - 1.0, mid + 1.0)
    with pytest.raises(sq.SQError, match="bounds too tight"):
        g.moments()


def test_fp64_batch_of_patch_ring_and_streamed_cubes():
    """25- and 31-point groups beside a 33-point one, whose odd-sized buffers set the
    distance between the workgroups' buffers."""
    from paper_1708_07913_amd import sq
    print("case FP64 batch of 25, 31 and 33 points", flush=True)
    wls = [W.fcc_workload("b25", 1, 7.78, 0.1, 3, 0.5, 6.0, 16, 1.0), W.fcc_workload("b31", 1, 7.78, 0.1, 4, 0.4, 6.0, 24, 1.0),
           W.fcc_workload("b33", 1, 8.0, 0.1, 24, 0.5, 8.0, 16, 1.0)]
    snaps = [sq.SQ.from_workload(wl, veff=torch.from_numpy(wl.veff()).cuda()) for wl in wls]
    ref = [g.scf_pass(wl.n_electrons) for g, wl in zip(snaps, wls)]
    ref = [(m.cpu().numpy(), mu, r.cpu().numpy(), e) for m, mu, r, e in ref]
    b = sq.Batch(snaps, [wl.n_electrons for wl in wls])
    assert sorted(b.groups()) == [(25, 1, 0), (31, 1, 0), (33, 1, 0)]
    for _ in range(3):
        mu, e = b.step()
        for i, (m1, mu1, r1, e1) in enumerate(ref):
            assert np.abs(b.moments[i].cpu().numpy() - m1).max() < 1e-12
            assert abs(mu[i] - mu1) < 1e-11
            assert np.abs(b.rho[i].cpu().numpy() - r1).max() < 1e-12 * r1.max()
            assert np.abs(e[i] - e1).max() < 1e-10 * np.abs(e1).max()
        torch.cuda.synchronize()


# cube side, chains: cell length, mesh, R_cut; 17 and 19 points with and without
# overlapping spheres (two rows per thread in FP64, one in mixed mode)
TWO_ROWS = {(17, 1): (9.0, 0.55, 4.4), (17, 2): (6.5, 0.5, 4.0), (19, 1): (8.0, 0.5, 4.5),
            (21, 2): (6.5, 0.5, 5.0), (21, 4): (6.0, 0.5, 5.0)}


@pytest.mark.parametrize("cube,chains", sorted(TWO_ROWS))
def test_two_row_cubes(cube, chains):
    from paper_1708_07913_amd import sq
    print(f"case {cube} points, {chains} chains", flush=True)
    a, h, rcut = TWO_ROWS[cube, chains]
    wl = W.fcc_workload(f"c{cube}", 1, a, 0.2, 3, h, rcut, 12, 1.0, fd_order=8 if cube == 17 else 12)
    V = wl.veff()
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda())
    assert_kernels(g, cube, chains)
    o = oracle.Oracle.from_workload(wl, veff=V)
    nodes = sample(g)
    compare(g, o, nodes)
    lo, hi = (t.cpu().numpy() for t in g.spectral_bounds())
    gm = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda(), precision=sq.FP32_MIXED)
    gm.set_bounds(torch.from_numpy(lo), torch.from_numpy(hi))
    mm = gm.moments().cpu().numpy()
    assert np.abs(mm[nodes] - o.moments(lo[nodes], hi[nodes], nodes=nodes)).max() < 1e-5
