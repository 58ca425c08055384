"""Guards of the patch kernels' build: the compiler flag they cannot do without, and
the scan of the generated code for vector instructions behind an empty execution
mask."""
from __future__ import annotations

import os
import subprocess

import pytest

from paper_1708_07913_amd import build

# a masked loop left with exec = 0, a constant written there, then the restore
LOOP = """\t.text
_Zkernel:
.LBB0_1:
\tds_add_f64 v1, v[2:3]
\ts_andn2_b64 exec, exec, s[0:1]
\ts_cbranch_execnz .LBB0_1
%s
\ts_or_b64 exec, exec, s[2:3]
\tv_lshlrev_b32_e32 v4, v33, v5
\ts_endpgm
"""
SKIP = """_Zkernel:
\ts_and_saveexec_b64 s[0:1], vcc
\ts_cbranch_execz .LBB0_2
\tv_add_f64 v[0:1], v[2:3], v[4:5]
.LBB0_2:
%s
\ts_or_b64 exec, exec, s[0:1]
\ts_endpgm
"""


@pytest.mark.parametrize("code", [LOOP, SKIP])
def test_scan_finds_writes_behind_an_empty_mask(code):
    assert build.masked_writes(code % "\tv_mov_b32_e32 v33, 3") != []
    assert build.masked_writes(code % "\ts_mov_b32 s4, 3 ; scalar") == []
    assert build.masked_writes(code % "\tv_readlane_b32 s4, v5, 1") == []


def test_patch_kernels_refuse_to_compile_without_the_flag():
    src = os.path.join(build.CSRC, "sq_tile_kernels.hip")
    cmd = [build.HIPCC, *build.DEVICE_FLAGS, "--cuda-device-only", "-E", src, "-o", os.devnull]
    flags = [f for f in build.TILE_FLAGS if f.startswith("-D")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode != 0 and "amdgpu-remove-redundant-endcf" in r.stderr
    assert subprocess.run([*cmd, *flags], capture_output=True).returncode == 0
    assert "-amdgpu-remove-redundant-endcf=0" in build.TILE_FLAGS
