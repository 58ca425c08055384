"""The benchmark's kernel names and hash: what it reports is what the workload runs."""
from __future__ import annotations

import pytest

import bench
from paper_1708_07913_amd import build
from paper_1708_07913_amd import workloads as W


def test_kernel_hash_covers_layouts_and_flags(monkeypatch, tmp_path):
    whole = bench.kernel_hash()
    names = [f.rsplit("/", 1)[1] for f in bench.KERNEL_SOURCES]
    assert {"sq_kernels.hip", "sq_tile_kernels.hip", "sq_device.h", "sq_internal.h"} <= set(names)
    monkeypatch.setattr(build, "TILE_FLAGS", [*build.TILE_FLAGS, "-O2"])
    assert bench.kernel_hash() != whole


# region, chains: kernels of an FP64 pass
CASES = {
    "patch29": ((7.78, 0.5, 7.0), "lanczos_tile_kernel", "moments_tile_kernel"),
    "ring31": ((6.0, 0.4, 5.9), "lanczos_ring_kernel", "moments_ring_kernel"),  # overlapping spheres
    "ring23": ((7.78, 0.5, 5.5), "lanczos_ring_kernel", "moments_ring_kernel"),
    "streamed33": ((8.0, 0.5, 8.0), "lanczos_kernel", "moments_kernel"),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_names_follow_the_dispatch(name):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07913_amd import sq
    (a, h, rcut), lanczos, moments = CASES[name]
    wl = W.fcc_workload(name, 1, a, 0.2, 3, h, rcut, 12, 1.0)
    g = sq.SQ.from_workload(wl, veff=torch.from_numpy(wl.veff()).cuda())
    names = [n for n, _ in bench.recurrence_kernels(g, wl.n_electrons)]
    assert names == [lanczos, moments]
