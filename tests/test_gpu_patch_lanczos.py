"""GPU parity of the patch kernels' Lanczos bounds (FP64, 25-31-point cubes,
spheres that do not overlap) against the FP64 CPU oracle where the kernel leaves
its usual path: potentials with high, narrow peaks, where alpha' is not small
beside beta and the sums are taken from the vector itself.

Tolerances, of the largest |eigenvalue|: the peaks make near-degenerate eigenvalues,
on which a long recurrence is ill-conditioned.  On the cells below the oracle is
within 1.1e-13 of its long-double form after 16 steps, hence 1e-12 there, and within
1.2e-6 after 50, hence 1e-4.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1708_07913_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# cube side: cell length, mesh, R_cut; overlap depth 1, mesh narrower (25: wider) than the cube
CELLS = {25: (8.4, 0.3, 3.6), 27: (7.78, 0.5, 6.5), 29: (7.78, 0.5, 7.0), 31: (7.78, 0.4, 6.0)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07913_amd import sq
    sq.load_library()
    torch.cuda.set_device(0)


def patch_cell(cube, npl=16, seed=5):
    a, h, rcut = CELLS[cube]
    return W.fcc_workload(f"c{cube}", 1, a, 0.1, seed, h, rcut, npl, 1.0)


def assert_patch_kernels(g, wl, cube):
    """One projector chain and the default shape: what the patch kernels serve."""
    from paper_1708_07913_amd import sq
    assert sq.Batch([g], [wl.n_electrons]).groups() == [(cube, 1, 0)]


@pytest.mark.parametrize("cube", sorted(CELLS))
@pytest.mark.parametrize("steps,tol", [(16, 1e-12), (50, 1e-4)])
def test_bounds_of_peaked_potential(cube, steps, tol):
    from paper_1708_07913_amd import sq
    print(f"case {cube} peaks, {steps} steps", flush=True)
    wl = patch_cell(cube)
    V = wl.veff()
    nodes = np.sort(np.random.default_rng(cube).choice(V.size, 24, replace=False))
    V[nodes[:8]] = 1e4
    V[nodes[8:12]] = -1e4
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda(), n_lanczos=steps)
    assert_patch_kernels(g, wl, cube)
    lo, hi = (t.cpu().numpy()[nodes] for t in g.spectral_bounds())
    lo_ref, hi_ref = oracle.Oracle.from_workload(wl, veff=V, n_lanczos=steps).bounds(nodes=nodes)
    scale = max(np.abs(lo_ref).max(), np.abs(hi_ref).max())
    assert np.abs(lo - lo_ref).max() < tol * scale
    assert np.abs(hi - hi_ref).max() < tol * scale


def test_one_step_at_the_range_of_doubles():
    """One Lanczos step has no beta: |u|^2 past the largest double is no error."""
    from paper_1708_07913_amd import sq
    wl = patch_cell(29)
    V = np.where(np.arange(wl.n ** 3) % 3 == 0, 1e160, -2e160)
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda(), n_lanczos=1)
    assert_patch_kernels(g, wl, 29)
    nodes = np.array([0, 1, 1234, g.nd - 1])
    lo, hi = (t.cpu().numpy()[nodes] for t in g.spectral_bounds())
    lo_ref, hi_ref = oracle.Oracle.from_workload(wl, veff=V, n_lanczos=1).bounds(nodes=nodes)
    assert np.isfinite(lo_ref).all()
    assert np.abs(lo - lo_ref).max() < 1e-12 * 2e160 and np.abs(hi - hi_ref).max() < 1e-12 * 2e160
