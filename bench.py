"""Benchmark: one SQ density/energy pass (SCF iteration at fixed V_eff) per step.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload large|paper|tiny|...]

A step runs every stage of the hot path on the resident inputs: Lanczos
spectral bounds -> Chebyshev moments -> Fermi level -> density and energies.
The default workload is the 1372-atom large cell (109^3 grid, 29^3 regions,
n_pl = 64, FP64), the configuration the FP64-versus-FP32-mixed seconds-per-SCF
metric is quoted on.  One JSON line is printed with the throughput in
grid-point x Chebyshev-step per second over whole steps, the roofline of the
dominant kernel (HIP events on the working stream), the FP32-mixed pass, the
errors of both precisions against the stored FP64 oracle results of the cell
(when present) and the FP64 CPU oracle timed on a bounded node sample.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

T_START = time.perf_counter()
ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "SQ grid-pt*Chebyshev-steps/s & s/SCF iter, FP64 vs FP32-mixed at rho err 1e-5"
HBM_PEAK_GBS = 8000.0
KERNEL_SOURCES = [os.path.join(ROOT, "paper_1708_07913_amd", "csrc", f)
                  for f in ("sq_kernels.hip", "sq_tile_kernels.hip", "sq_device.h", "sq_internal.h")]


def log(msg: str) -> None:
    """Progress line on stderr, with seconds since the bench started."""
    print(f"[bench {time.perf_counter() - T_START:7.1f}s] {msg}", file=sys.stderr, flush=True)


def kernel_hash() -> str:
    """Hash of the kernel code (device sources, the header with their layouts and
    dispatch rules, compiler flags) with comments and whitespace removed, so that a
    comment edit keeps the recorded counter traffic valid."""
    import re

    from paper_1708_07913_amd import build
    text = "\n".join(open(f).read() for f in KERNEL_SOURCES)
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    text = " ".join(text.split() + build.DEVICE_FLAGS + build.TILE_FLAGS)
    return hashlib.sha256(text.encode()).hexdigest()[:16]


FP64_VALU_TFLOPS = 78.6
FLOPS_PER_POINT = 44  # 37-point stencil as pair sums, centre/V, -t^{k-1}


def copy_bandwidth(torch, nbytes: int = 1 << 30, reps: int = 5) -> float:
    """HBM bandwidth of a device-to-device copy (bytes read + written per second),
    median of `reps` copies timed with events on the current stream."""
    src = torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(1)
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    times = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        dst.copy_(src)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e-3)
    del src, dst
    return 2.0 * nbytes / float(np.median(times))


def stencil_roofline(bytes_, flops, seconds, bw):
    """T_roof / T with T_roof = max(bytes / measured copy bandwidth, flops / FP64 VALU peak)."""
    t_roof = max(bytes_ / bw, flops / (FP64_VALU_TFLOPS * 1e12))
    return {"t_roof_s": t_roof, "t_s": seconds, "frac": t_roof / seconds,
            "algorithmic_bytes": bytes_, "flops": flops}


# planes of the previous vector that the patch kernels keep in LDS (Lanczos, moments)
PATCH_LDS_PLANES = {25: (10, 10), 27: (9, 10), 29: (8, 9), 31: (8, 8)}


def recurrence_kernels(g, n_electrons):
    """((name, words), ...) of the FP64 Lanczos and moments kernels of a context: the
    words per region point and step that stream through the workgroup's buffers.
    Patch kernels (25-31 points, one projector chain): the previous vector in and
    out, but for the planes in LDS.  Ring kernels (up to 31 points): Lanczos x_{j-1}
    and x_{j-2} in and x_j out, moments t^{k-1} in and t^k out.  Streamed kernels:
    three each."""
    from paper_1708_07913_amd import sq
    (C, chains, _), = sq.Batch([g], [n_electrons], use_graph=False).groups()
    if C in PATCH_LDS_PLANES and chains == 1:
        return tuple((f"{k}_tile_kernel", 2.0 * (C - p) / C)
                     for k, p in zip(("lanczos", "moments"), PATCH_LDS_PLANES[C]))
    if C <= 31:
        return ("lanczos_ring_kernel", 3.0), ("moments_ring_kernel", 2.0)
    return ("lanczos_kernel", 3.0), ("moments_kernel", 3.0)


def workload(name):
    from paper_1708_07913_amd import workloads as W
    return {"paper": W.paper_size_cell, "paper-small": W.paper_cell_small, "large": W.large_cell,
            "tiny": W.tiny_cell}[name]()


def traffic_from_profiles(kernel_key: str, workload_name: str):
    """HBM bytes per launch from committed rocprofv3 counter summaries, only if
    they were taken on the current kernel source."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        data = json.load(open(path))
        ent = data.get(f"{kernel_key}:{workload_name}")
        if ent and ent.get("kernel_source_sha") == kernel_hash():
            return ent["bytes_per_launch"]
    except (ValueError, KeyError):
        return None
    return None


def run_gpu(wl, steps, warmup, precision):
    """W untimed and K timed full passes; per-phase times from HIP events on
    the stream the library launches on (torch's current stream)."""
    import torch
    from paper_1708_07913_amd import sq

    V = torch.from_numpy(wl.veff()).cuda()
    g = sq.SQ.from_workload(wl, veff=V, precision=precision)
    stream = torch.cuda.current_stream()
    tag = "fp64" if precision == sq.FP64 else "mixed"
    log(f"{tag}: context ready, {warmup} warm-up pass(es)")
    for w in range(warmup):
        g.scf_pass(wl.n_electrons)
        log(f"{tag}: warm-up {w + 1}/{warmup} done")
    torch.cuda.synchronize()
    log(f"{tag}: {steps} timed pass(es)")
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(5)] for _ in range(steps)]
    out = None
    t0 = time.perf_counter()
    for s in range(steps):
        e = ev[s]
        e[0].record(stream)
        bounds = g.spectral_bounds()
        e[1].record(stream)
        mom = g.moments()
        e[2].record(stream)
        mu = g.fermi_level(mom, wl.n_electrons)
        e[3].record(stream)
        rho, en = g.density_energy(mom, mu)
        e[4].record(stream)
        out = (bounds, mom, mu, rho, en)
        # the Fermi search has read back its counts, so this step's moments
        # are done; a line per step shows progress on long runs
        log(f"{tag}: step {s + 1}/{steps} mu {mu:.12f}")
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    phases = np.array([[ev[s][i].elapsed_time(ev[s][i + 1]) for i in range(4)] for s in range(steps)])
    return g, out, wall, phases.mean(0)  # ms per phase


def reuse_pass(g, bounds, n_electrons):
    """One SCF pass that reuses the previous pass's bounds (re-injected with
    sq_set_bounds), timed on the host around the synchronising calls."""
    import torch
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    g.set_bounds(*bounds)
    mom = g.moments()
    mu = g.fermi_level(mom, n_electrons)
    g.density_energy(mom, mu)
    torch.cuda.synchronize()
    return time.perf_counter() - t0


def projector_nodes(wl) -> int:
    """Grid nodes inside at least one projector sphere (|x - R| <= r_c on the
    periodic grid): the nodes that carry nonlocal force contributions."""
    from paper_1708_07913_amd import workloads as W
    n = W.grid_points_per_axis(wl.cell, wl.h)
    h = wl.cell / n
    hit = np.zeros(n ** 3, dtype=bool)
    for R, (_, rc, _) in zip(np.asarray(wl.atoms, float), np.asarray(wl.kb, float)):
        r = int(np.ceil(rc / h)) + 1
        b = np.floor(R / h).astype(int)
        d = np.arange(-r, r + 2)
        ii, jj, kk = np.meshgrid(b[0] + d, b[1] + d, b[2] + d, indexing="ij")
        pts = np.stack([ii.ravel(), jj.ravel(), kk.ravel()], 1)
        inside = (((pts * h - R) ** 2).sum(1) <= rc * rc)
        loc = np.mod(pts[inside], n)
        hit[loc[:, 0] + n * (loc[:, 1] + n * loc[:, 2])] = True
    return int(hit.sum())


def forces_leg(g, wl, mu):
    """One sq_nl_forces call (nonlocal forces, recurrence to n_pl) at the last
    pass's bounds and Fermi level, timed on the host around the synchronising
    call."""
    t0 = time.perf_counter()
    F = g.nl_forces(mu)
    sec = time.perf_counter() - t0
    nodes = projector_nodes(wl)
    C = 2 * g.m + 1
    node_steps = nodes * wl.npl
    # per node-step: t^k, t^{k-1} in, t^{k+1} out, u in and out
    nbytes = node_steps * 5 * C ** 3 * 8
    return {"seconds": sec, "nodes": nodes, "node_steps": node_steps, "node_steps_per_s": node_steps / sec,
            "algorithmic_bytes": nbytes, "achieved_GBs": nbytes / sec / 1e9,
            "max_abs_force_Ha_per_bohr": float(np.abs(F).max())}


def golden_path(wl):
    names = {"al256_h0.4_rc6": "paper", "al1372_h0.5_rc7": "large"}
    if wl.name not in names:
        return None
    path = os.path.join(ROOT, "tests", "golden", f"full_{names[wl.name]}.npz")
    return path if os.path.exists(path) else None


def accuracy_vs_oracle(wl, ctx, path):
    """Errors of one context against the stored FP64 oracle results of the
    whole cell: the oracle's bounds are injected, the moments, Fermi level,
    density and energies recomputed on the GPU and compared at the oracle's
    Fermi level (rho at the stored nodes, energies of the whole cell)."""
    import json as _json
    import torch
    with np.load(path, allow_pickle=False) as z:
        d = {k: z[k] for k in z.files}
    q = _json.loads(str(d["meta"]))["qscale"]
    ctx.set_bounds(torch.from_numpy(d["qlo"].astype(np.float64) / q),
                   torch.from_numpy(d["qhi"].astype(np.float64) / q))
    mom = ctx.moments()
    mu = ctx.fermi_level(mom, wl.n_electrons)
    rho, e = ctx.density_energy(mom, float(d["mu"]))
    r = rho.cpu().numpy()[d["rho_nodes"]]
    _, e_own = ctx.density_energy(mom, mu)
    eo = d["energies"]
    return {"rho_max_rel_err": float(np.abs(r - d["rho"]).max() / float(d["rho_max"])),
            "E_band_err_Ha_per_atom": float(abs(e_own[0] - eo[0]) / wl.natom),
            "F_err_Ha_per_atom": float(abs(e_own[2] - eo[2]) / wl.natom),
            "electron_count_err": float(abs(e_own[3] - wl.n_electrons)),
            "mu_err_Ha": float(abs(mu - float(d["mu"]))),
            "at_oracle_mu": {"E_band_err_Ha_per_atom": float(abs(e[0] - eo[0]) / wl.natom),
                             "F_err_Ha_per_atom": float(abs(e[2] - eo[2]) / wl.natom),
                             "electron_count_diff": float(e[3] - eo[3])},
            "reference": "stored FP64 oracle results of the whole cell (oracle bounds injected); rho at "
                         f"{r.size} nodes at the oracle's mu, energies at each side's own mu"}


def tuner_entry(cache, precision_tag, groups):
    """The autotuner's cache entry for this batch signature (precision and the
    (cube, chains) of its launch groups), or None."""
    try:
        data = json.load(open(cache))
    except (OSError, ValueError):
        return None
    want = {(c, k) for c, k, _ in groups}
    for key, val in data.items():
        parts = key.split("/")
        if "lms" not in parts or parts[parts.index("lms") + 1] != precision_tag:
            continue
        have = set()
        for p in parts[parts.index("lms") + 2:]:
            ck = p.split(":")[0]
            have.add((int(ck[1:].split("x")[0]), int(ck.split("x")[1])))
        if have == want:
            return val
    return None


def run_ensemble(args):
    """The 12-snapshot QMD ensemble as one batch (persistent work-queue launches,
    device Brent, hipGraph replay), tiles autotuned on the first call."""
    import tempfile

    import torch
    from paper_1708_07913_amd import sq
    from paper_1708_07913_amd import workloads as W

    wls = W.qmd_ensemble()
    prec = sq.FP64 if args.precision == "fp64" else sq.FP32_MIXED
    snaps = [sq.SQ.from_workload(wl, veff=torch.from_numpy(wl.veff()).cuda(), precision=prec) for wl in wls]
    b = sq.Batch(snaps, [wl.n_electrons for wl in wls], use_graph=True)
    cache = os.environ.get("SQ_TILE_CACHE", os.path.join(tempfile.gettempdir(), "sq_tiles.json"))
    t0 = time.perf_counter()
    tiles = b.autotune(cache)
    tune_s = time.perf_counter() - t0
    # kernel shape bits per launch group (1: two rows per thread, 2: two planes per barrier)
    tiles["shapes"] = [list(g) for g in b.groups()]
    entry = tuner_entry(cache, "fp64" if prec == sq.FP64 else "mixed", b.groups())
    if entry is not None:
        # sample time (ms) per group at shape bits 0..3 (-1: shape absent)
        tiles["shape_ms"] = entry.get("shape_ms")
    log(f"ensemble: tiles {tiles} ({tune_s:.1f} s)")
    for _ in range(args.warmup):
        b.step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        mu, e = b.step()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    log(f"ensemble: {args.steps} timed pass(es), {wall / args.steps:.2f} s per pass")
    # SCF-style passes that reuse the bounds of the previous pass
    br = sq.Batch(snaps, [wl.n_electrons for wl in wls], use_graph=True, bounds_every=1000)
    br.step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    br.step()
    torch.cuda.synchronize()
    reuse_s = time.perf_counter() - t1
    del br
    log(f"ensemble: pass reusing bounds {reuse_s:.2f} s")
    # the same pass with the default tiles (32 nodes per item, occupancy-limited
    # workgroups per CU, default kernel shapes), for the autotuner's gain
    bd = sq.Batch(snaps, [wl.n_electrons for wl in wls], use_graph=True)
    bd.step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    bd.step()
    torch.cuda.synchronize()
    default_s = time.perf_counter() - t1
    default_tiles = bd.tiles()
    default_tiles["shapes"] = [list(g) for g in bd.groups()]
    del bd
    log(f"ensemble: default tiles {default_tiles}: {default_s:.2f} s per pass")
    node_steps = sum(g.nd * (wl.npl // 2) for g, wl in zip(snaps, wls))
    nodes = sum(g.nd for g in snaps)
    rec = {"metric": METRIC, "value": node_steps / (wall / args.steps), "unit": "grid-pt*Chebyshev-steps/s",
           "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": 1e3 * wall / args.steps,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "f64" if prec == sq.FP64 else "f32-storage/f64-accumulate",
           "data": "synthetic (12 seeded FCC Al-like snapshots, Gaussian-well V_eff, s-type KB projectors)",
           "config": {"workload": "qmd_ensemble_12", "snapshots": len(wls), "n_nodes": nodes,
                      "cubes": sorted({2 * g.m + 1 for g in snaps}), "npl": sorted({wl.npl for wl in wls}),
                      "parallelism": "single GPU", "batch": "one persistent launch per cube size, hipGraph"},
           "s_per_scf": wall / args.steps, "s_per_scf_reusing_bounds": reuse_s, "tiles": tiles,
           "autotune_s": tune_s, "s_per_scf_default_tiles": default_s, "default_tiles": default_tiles,
           "electron_count_err_max": float(max(abs(e[i][3] - wl.n_electrons) for i, wl in enumerate(wls)))}
    if prec == sq.FP32_MIXED:
        # error of the mixed recurrence per snapshot, against the FP64 path on the
        # same (FP64) bounds and at the batch's Fermi level
        errs = []
        for i, (wl, gm) in enumerate(zip(wls, snaps)):
            g64 = sq.SQ.from_workload(wl, veff=torch.from_numpy(wl.veff()).cuda(), precision=sq.FP64)
            lo, hi = g64.spectral_bounds()
            mom64 = g64.moments()
            gm.set_bounds(lo, hi)
            rho64, e64 = g64.density_energy(mom64, float(mu[i]))
            rhom, em = gm.density_energy(gm.moments(), float(mu[i]))
            r64, rm = rho64.cpu().numpy(), rhom.cpu().numpy()
            errs.append({"snapshot": wl.name, "rho_max_rel_err": float(np.abs(rm - r64).max() / r64.max()),
                         "E_band_err_Ha_per_atom": float(abs(em[0] - e64[0]) / wl.natom),
                         "F_err_Ha_per_atom": float(abs(em[2] - e64[2]) / wl.natom)})
            log(f"{wl.name}: mixed rho err {errs[-1]['rho_max_rel_err']:.2e}")
            del g64, mom64, rho64, rhom
        rec["mixed_vs_fp64"] = {"rho_max_rel_err": max(x["rho_max_rel_err"] for x in errs),
                                "E_band_err_Ha_per_atom": max(x["E_band_err_Ha_per_atom"] for x in errs),
                                "F_err_Ha_per_atom": max(x["F_err_Ha_per_atom"] for x in errs),
                                "per_snapshot": errs}
    print(json.dumps(rec), flush=True)


def run_mixed_sweep():
    """FP32-mixed against the FP64 path on the tiny cell for kT in {0.5, 1, 2, 5} eV
    and n_pl in {32, 48, 96}: the FP64 bounds and Fermi level are injected, so the
    errors are those of the mixed recurrence alone (the FP64 path itself matches
    the oracle to 1e-10 in the parity tests)."""
    import torch
    from paper_1708_07913_amd import sq
    from paper_1708_07913_amd import workloads as W

    rows = []
    for kT in (0.5, 1.0, 2.0, 5.0):
        for npl in (32, 48, 96):
            wl = W.tiny_cell("mixed", npl=npl, kT_eV=kT)
            V = torch.from_numpy(wl.veff()).cuda()
            g = sq.SQ.from_workload(wl, veff=V, precision=sq.FP64)
            mom, mu, rho64, e64 = g.scf_pass(wl.n_electrons)
            lmin, lmax = g.spectral_bounds()
            gm = sq.SQ.from_workload(wl, veff=V, precision=sq.FP32_MIXED)
            gm.set_bounds(lmin, lmax)
            rho, e = gm.density_energy(gm.moments(), mu)
            torch.cuda.synchronize()
            r, r64 = rho.cpu().numpy(), rho64.cpu().numpy()
            rows.append({"kT_eV": kT, "npl": npl,
                         "rho_max_rel_err": float(np.abs(r - r64).max() / r64.max()),
                         "E_band_err_Ha_per_atom": float(abs(e[0] - e64[0]) / wl.natom),
                         "F_err_Ha_per_atom": float(abs(e[2] - e64[2]) / wl.natom),
                         "electron_count_err": float(abs(e[3] - e64[3]))})
            log(f"mixed sweep kT={kT} npl={npl}: {rows[-1]}")
    print(json.dumps({"workload": "al4_h0.5_rc2.5 mixed-precision sweep", "reference": "FP64 GPU path",
                      "rows": rows, "max_rho_rel_err": max(x["rho_max_rel_err"] for x in rows)}), flush=True)


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def cpu_baseline(wl, budget_s=12.0):
    """The FP64 oracle on a bounded node sample of the same workload (bounds +
    moments, the per-node work of a step), scaled to node-steps per second."""
    import oracle
    V = wl.veff()
    o = oracle.Oracle.from_workload(wl, veff=V)
    rng = np.random.default_rng(0)
    count, elapsed = 8, 0.0
    while True:
        nodes = rng.choice(o.nd, count, replace=False)
        t = time.perf_counter()
        lo, hi = o.bounds(nodes)
        o.moments(lo, hi, nodes=nodes)
        elapsed = time.perf_counter() - t
        if elapsed >= budget_s / 2 or count >= o.nd:
            break
        count = int(min(o.nd, max(2 * count, count * (budget_s / 1.5) / max(elapsed, 1e-3))))
    rate = count * (wl.npl // 2) / elapsed
    return {"value": rate, "unit": "grid-pt*Chebyshev-steps/s", "cores": oracle.num_threads(),
            "cpu_model": cpu_model(), "kind": "oracle",
            "sample": f"{count} random nodes of {o.nd} (seed 0): Lanczos bounds + moments, {elapsed:.1f} s"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="large",
                    choices=["large", "paper", "paper-small", "tiny", "ensemble", "mixed-sweep"])
    ap.add_argument("--precision", default="mixed", choices=["fp64", "mixed"],
                    help="precision of the ensemble workload")
    ap.add_argument("--mixed-steps", type=int, default=1, help="timed FP32-mixed passes")
    ap.add_argument("--mixed-warmup", type=int, default=0,
                    help="untimed FP32-mixed passes")
    ap.add_argument("--no-mixed", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-accuracy", action="store_true")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a 1 GiB device-to-device copy (counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this implementation runs on one GPU; --gpus must be 1",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    from paper_1708_07913_amd import sq
    log("torch imported")

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        sys.exit(2)
    torch.cuda.set_device(0)
    if args.copy_calibration:
        src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
        log("copy calibration: 1 GiB device-to-device")
    if args.workload == "ensemble":
        run_ensemble(args)
        return
    if args.workload == "mixed-sweep":
        run_mixed_sweep()
        return
    wl = workload(args.workload)
    log(f"{wl.name}: n={wl.n} natom={wl.natom} npl={wl.npl}")

    g, (bounds, mom, mu, rho, en), wall, ph = run_gpu(wl, args.steps, args.warmup, sq.FP64)
    nd, S = g.nd, wl.npl // 2
    C = 2 * g.m + 1
    ns = C ** 3
    ms_step = 1e3 * wall / args.steps
    value = nd * S / (wall / args.steps)
    log(f"fp64: {ms_step:.1f} ms/step phases(ms) bounds {ph[0]:.1f} moments {ph[1]:.1f} "
          f"fermi {ph[2]:.1f} density {ph[3]:.1f}")
    reuse_s = reuse_pass(g, bounds, wl.n_electrons)
    log(f"pass reusing bounds: {reuse_s:.2f} s")
    forces = None
    if wl.npl <= 256:
        forces = forces_leg(g, wl, mu)
        log(f"nonlocal forces: {forces['seconds']:.2f} s over {forces['nodes']} nodes")

    # the dominant kernel against the nearer roof: the bytes it streams at the HBM peak,
    # or the algorithmic FP64 operations at the vector peak
    (lname, lwords), (mname, mwords) = recurrence_kernels(g, wl.n_electrons)
    lanczos_bytes = nd * 50 * lwords * ns * 8
    moments_bytes = nd * S * mwords * ns * 8
    flops_step = nd * ns * FLOPS_PER_POINT
    if ph[0] >= ph[1]:
        kname, kbytes, kflops, kms = lname, lanczos_bytes, 50 * flops_step, ph[0]
    else:
        kname, kbytes, kflops, kms = mname, moments_bytes, S * flops_step, ph[1]
    if kbytes / (HBM_PEAK_GBS * 1e9) >= kflops / (FP64_VALU_TFLOPS * 1e12):
        bound, achieved, peak, unit = "hbm", kbytes / (kms * 1e-3) / 1e9, HBM_PEAK_GBS, "GB/s"
    else:
        bound, achieved, peak, unit = "fp64", kflops / (kms * 1e-3) / 1e12, FP64_VALU_TFLOPS, "TFLOP/s"
    roof = {"bound": bound, "achieved": achieved, "peak": peak, "unit": unit,
            "frac": achieved / peak, "traffic": traffic_from_profiles(kname, wl.name),
            "kernel": kname, "algorithmic_bytes_per_launch": kbytes, "flops_per_launch": kflops,
            "avg_launch_ms": kms}

    bw = copy_bandwidth(torch)
    roof_meas = {"bw_measured_GBs": bw / 1e9,
                 "bw_source": "1 GiB device-to-device copy (read + write bytes), median of 5",
                 "fp64_valu_peak_TFLOPs": FP64_VALU_TFLOPS,
                 "lanczos": stencil_roofline(lanczos_bytes, 50 * flops_step, ph[0] * 1e-3, bw),
                 "moments_fp64": stencil_roofline(moments_bytes, S * flops_step, ph[1] * 1e-3, bw)}

    rec = {"metric": METRIC, "value": value, "unit": "grid-pt*Chebyshev-steps/s", "n_gpus": 1,
           "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
           "data": "synthetic (seeded FCC Al-like cell, Gaussian-well V_eff, s-type KB projectors)",
           "config": {"workload": wl.name, "n_grid": wl.n, "n_nodes": nd, "region_points": ns,
                      "npl": wl.npl, "n_lanczos": 50, "natom": wl.natom, "kT_eV": wl.kT_eV,
                      "parallelism": "single GPU"},
           "s_per_scf": wall / args.steps,
           # measured: bounds of the previous pass re-injected, then moments,
           # Fermi level, density and energies
           "s_per_scf_reusing_bounds": reuse_s,
           "moments_node_steps_per_s": nd * S / (ph[1] * 1e-3),
           "phase_ms": {"bounds": ph[0], "moments": ph[1], "fermi": ph[2], "density": ph[3]},
           "roofline": roof,
           # the same kernels against the bandwidth a plain copy reaches on this GPU
           "stencil_roofline_measured_bw": roof_meas,
           "electron_count": float(en[3]), "mu": mu}
    if forces is not None:
        rec["nl_forces"] = forces
    del mom, rho

    gm = None
    if not args.no_mixed:
        gm, (_, _, _, _, en_m), wall_m, ph_m = run_gpu(wl, args.mixed_steps, args.mixed_warmup,
                                                        sq.FP32_MIXED)
        rec["mixed"] = {"steps": args.mixed_steps, "warmup": args.mixed_warmup,
                        "ms_per_step": 1e3 * wall_m / args.mixed_steps,
                        "value": nd * S / (wall_m / args.mixed_steps),
                        "moments_node_steps_per_s": nd * S / (ph_m[1] * 1e-3),
                        "phase_ms": {"bounds": ph_m[0], "moments": ph_m[1], "fermi": ph_m[2],
                                     "density": ph_m[3]},
                        "electron_count_err": float(abs(en_m[3] - wl.n_electrons))}
        # FP32 storage; up to 31 points always a ring kernel (two words), beyond them the FP64 one
        mixed_bytes = nd * S * 2 * ns * 4 if C <= 31 else moments_bytes
        roof_meas["moments_mixed"] = stencil_roofline(mixed_bytes, S * flops_step, ph_m[1] * 1e-3, bw)
        log(f"mixed: {rec['mixed']['ms_per_step']:.1f} ms/step")

    path = golden_path(wl)
    if path and not args.no_accuracy:
        acc = {"fp64": accuracy_vs_oracle(wl, g, path)}
        if gm is not None:
            acc["mixed"] = accuracy_vs_oracle(wl, gm, path)
        rec["accuracy_vs_oracle"] = acc
        log(f"accuracy vs oracle: {json.dumps(acc)}")

    if not args.no_cpu:
        rec["cpu_baseline"] = cpu_baseline(wl)
        log(f"cpu baseline: {rec['cpu_baseline']['sample']}")
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
