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
