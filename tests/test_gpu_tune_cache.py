"""Autotuner cache entries: what an entry of another kernel generation does, and
shape bits behind which a cube side has the same kernels."""
from __future__ import annotations

import json
import re

import pytest

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


def _batch(*wls):
    from paper_1708_07913_amd import sq
    snaps = [sq.SQ.from_workload(wl, veff=torch.from_numpy(wl.veff()).cuda()) for wl in wls]
    return sq.Batch(snaps, [wl.n_electrons for wl in wls])


def test_entries_without_the_generation_are_tuned_anew(tmp_path):
    """An entry under the untagged key (its shapes and tile were chosen for other
    kernels) is left alone and a new one is written beside it."""
    wl = W.fcc_workload("c25", 1, 8.4, 0.1, 5, 0.3, 3.6, 16, 1.0)
    cache = str(tmp_path / "tiles.json")
    _batch(wl).autotune(cache)
    (key, entry), = json.load(open(cache)).items()
    old = re.sub(r"/lms[^/]*/", "/lms/", key)
    entry.update(block_nodes=48, shapes=[[c, k, 3] for c, k, _ in entry["shapes"]])
    json.dump({old: entry}, open(cache, "w"))
    t = _batch(wl).autotune(cache)
    assert t["block_nodes"] in (8, 32, 128)
    data = json.load(open(cache))
    assert data[old] == entry and len(data) == 2


@pytest.mark.parametrize("precision,same", [("fp64", [(0, 1), (0, 3)]), ("mixed", [(1, 3)])])
def test_shapes_with_the_same_kernels_are_timed_once(tmp_path, precision, same):
    """21-point cubes: the two-row build is the FP64 default and has one plane a
    barrier.  Shape bits with the same kernels share one sample time (a second
    measurement hardly ever gives the same microseconds)."""
    wl = W.fcc_workload("c21", 2, 7.78, 0.1, 31, 0.5, 5.0, 24, 1.0, precision=precision)
    cache = str(tmp_path / "tiles.json")
    _batch(wl).autotune(cache)
    (entry,) = json.load(open(cache)).values()
    (cube, _, *ms), = entry["shape_ms"]
    assert cube == 21 and all(t > 0 for t in ms)
    assert all(ms[a] == ms[b] for a, b in same), ms
    assert entry["shapes"][0][2] not in [b for _, b in same]
