"""Rounding error of the FP64 moments of 25-31-point cubes against a long-double
recurrence on the same bounds.

Tolerance on the root-mean-square error of 24 nodes' moments (|moment| <= 1): one
unit roundoff 2^-53 for the cells as they are, and two where V_eff is 50 times as
deep (the diagonal, -75 to 20 Ha, then outweighs the stencil's legs).  The ring
kernels, which add the diagonal last, reach 0.8-0.9 and 1.35; adding it first
costs 0.9-1.5 and 3.3.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1708_07913_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CELLS = {25: (8.4, 0.3, 3.6), 27: (7.78, 0.5, 6.5), 29: (7.78, 0.5, 7.0), 31: (7.78, 0.4, 6.0)}
LD = np.longdouble


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07913_amd import sq
    sq.load_library()
    torch.cuda.set_device(0)


def long_double_moments(o, wl, V, q, lmin, lmax, margin=0.05):
    """Moments of node q by the recurrence in long double (weights, projector values
    and V_eff are the FP64 ones)."""
    n, m, npl = o.n, o.m, wl.npl
    C, no = 2 * m + 1, wl.fd_order // 2
    w = oracle.fd_weights(wl.fd_order, o.h).astype(LD)
    lo = np.array([q % n, (q // n) % n, q // (n * n)]) - m
    ax = [(lo[k] + np.arange(C)) % n for k in range(3)]
    diag = V.reshape(n, n, n)[np.ix_(ax[2], ax[1], ax[0])].astype(LD) - 3 * w[0]
    images = []
    for a in range(len(wl.atoms)):
        ijk, p = o.atom_table(a)
        reach = [range(-((lo[k] - ijk[:, k].max()) // -n) - 1, (lo[k] + C - 1 - ijk[:, k].min()) // n + 2) for k in range(3)]
        for tz in reach[2]:
            for ty in reach[1]:
                for tx in reach[0]:
                    x = ijk + n * np.array([tx, ty, tz]) - lo
                    inside = ((x >= 0) & (x < C)).all(1)
                    if inside.any():
                        images.append(((x[inside, 2], x[inside, 1], x[inside, 0]), p[inside].astype(LD),
                                       LD(wl.kb[a, 2]) * LD(o.h) ** 3))

    def apply(t):
        y = diag * t
        for k in range(3):
            for d in range(1, no + 1):
                hi, low = [slice(None)] * 3, [slice(None)] * 3
                hi[k], low[k] = slice(d, None), slice(None, -d)
                y[tuple(hi)] += LD(-0.5) * w[d] * t[tuple(low)]
                y[tuple(low)] += LD(-0.5) * w[d] * t[tuple(hi)]
        for at, p, c in images:
            y[at] += c * (p * t[at]).sum() * p
        return y

    chi, zeta = (LD(lmax) + LD(lmin)) / 2, LD(1 + margin) * (LD(lmax) - LD(lmin)) / 2
    t0 = np.zeros((C, C, C), dtype=LD)
    t0[m, m, m] = 1
    t1 = (apply(t0) - chi * t0) / zeta
    out = np.zeros(npl + 1, dtype=LD)
    out[0], half = 1, npl // 2
    first = t1[m, m, m]
    for k in range(1, half + 1):
        out[k] = t1[m, m, m]
        if k > half // 2:
            out[2 * k] = 2 * (t1 * t1).sum() - 1
            out[2 * k - 1] = 2 * (t1 * t0).sum() - first
        t0, t1 = t1, 2 * (apply(t1) - chi * t1) / zeta - t0
    return out


@pytest.mark.parametrize("cube", sorted(CELLS))
@pytest.mark.parametrize("depth,units", [(1.0, 1.0), (50.0, 2.0)])
def test_moments_against_long_double(cube, depth, units):
    from paper_1708_07913_amd import sq
    print(f"case {cube} V_eff x {depth}", flush=True)
    a, h, rcut = CELLS[cube]
    wl = W.fcc_workload(f"c{cube}", 1, a, 0.1, 5, h, rcut, 32, 1.0)
    V = depth * wl.veff()
    o = oracle.Oracle.from_workload(wl, veff=V)
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(V).cuda())
    assert sq.Batch([g], [wl.n_electrons]).groups() == [(cube, 1, 0)]  # the patch kernels' case
    lo, hi = (t.cpu().numpy() for t in g.spectral_bounds())
    nodes = np.random.default_rng(cube).choice(g.nd, 24, replace=False)
    g.set_bounds(lo, hi)
    m = g.moments().cpu().numpy()[nodes]
    ref = np.stack([long_double_moments(o, wl, V, int(q), lo[q], hi[q]) for q in nodes])
    rms = float(np.sqrt(np.mean((m - ref) ** 2)))
    print(f"  rms {rms / 2.0 ** -53:.2f} unit roundoffs", flush=True)
    assert rms < units * 2.0 ** -53
