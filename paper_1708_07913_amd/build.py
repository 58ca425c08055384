"""Build libsq.so (HIP kernels for gfx950 + the C ABI host code) in-tree.

The host code is plain C++ compiled by g++ against the HIP runtime API.

    python -m paper_1708_07913_amd.build

The kernels are compiled with packed FP32 instructions disabled; the host file
is compiled without floating-point contraction (the projector sphere test
r^2 <= r_c^2 must be evaluated exactly as written).
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsq.so")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DEVICE_FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
                "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-munsafe-fp-atomics",
                # the plane loops of the recurrence kernels must unroll fully
                # (register-resident columns are indexed by plane)
                "-mllvm", "-pragma-unroll-threshold=1000000"]
# optional extra -D definitions for the kernels (tuning knobs, e.g.
# "SQ_MOMENTS_AHEAD=3 SQ_LANCZOS_AHEAD=3")
DEVICE_FLAGS += ["-D" + d for d in os.environ.get("SQ_DEVICE_DEFINES", "").split()]
HOST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
              "-I/opt/rocm/include"]
CXX = os.environ.get("CXX", "g++")

# recurrence kernels are split into several translation units by cube size so
# that the build parallelises
CUBE_GROUPS = [[3, 5, 7, 9, 11, 13], [15, 17, 19], [21], [23], [25], [27], [29], [31], [33], [35], [37]]
# the two-row kernels of the 17-27-point cubes: a second build of the same
# source (SQ_TWO_ROWS=1, kernels in namespace sq::two_rows)
TWO_ROW_GROUPS = [[17, 19], [21], [23], [25], [27]]
# Patch kernels (sq_tile_kernels.hip).  Every end of a branch restores the
# execution mask by itself: with the compiler's pass that merges such ends, a
# constant that was rematerialised after a masked loop fell in front of the
# merged restore, was written with an empty mask, and a wild LDS address followed.
# The source does not compile without the macro; the pattern itself is looked for in
# the generated code of every kernel (masked_writes).
TILE_CUBES = [25, 27, 29, 31]
TILE_FLAGS = ["-mllvm", "-amdgpu-remove-redundant-endcf=0", "-DSQ_KEEP_BRANCH_ENDS"]


def masked_writes(listing: str) -> list[str]:
    """Vector instructions of an AMDGPU listing that stand between a point which can
    be reached with an empty execution mask (the way out of a masked loop, the target
    of an s_cbranch_execz) and the next write of the mask."""
    lines = listing.split("\n")
    # Branches that depend on the mask stand behind the instruction that may empty it.
    # (Others, in uniform regions, only mark a way that is always or never taken.)
    mask = r"^\s*s_\w*(?:saveexec\w* .*|\w+ exec,.*)\n\s*s_cbranch_exec"
    skipped_to = set(re.findall(mask + r"z (\S+)", listing, re.M))
    ways_back = {listing.count("\n", 0, m.end()) + 1 for m in re.finditer(mask + "nz", listing, re.M)}
    found, labels, empty = [], set(), False
    for number, line in enumerate(lines, 1):
        label = re.match(r"(\S+):", line)
        if label:
            if label.group(1).startswith(".LBB"):
                labels.add(label.group(1))
                empty = empty or label.group(1) in skipped_to
            else:
                labels, empty = set(), False
            continue
        text = line.split(";")[0].split()
        if not text:
            continue
        op, rest = text[0], text[1:]
        if number in ways_back and rest[0] in labels:
            empty = True
        elif "saveexec" in op or op in ("s_branch", "s_endpgm", "s_cbranch_execz") or \
                (op.startswith("s_") and rest and rest[0].startswith("exec")):
            empty = False
        elif empty and re.match(r"(v_(?!readlane|writelane|readfirstlane)|ds_|buffer_|global_|flat_|scratch_)", op):
            found.append(f"{number}: {' '.join(text)}")
    return found


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("command failed: " + " ".join(cmd))
    return r


def _compile(cmd, obj):
    """Compile one object; the listing of its device code, if there is one, must pass
    masked_writes."""
    tmp = obj + ".dir"
    os.makedirs(tmp, exist_ok=True)
    r = _run([*cmd, "-save-temps=obj", "-c", "-o", os.path.join(tmp, "out.o")])
    for name in os.listdir(tmp):
        if name.endswith(f"{ARCH}.s"):
            with open(os.path.join(tmp, name)) as f:
                found = masked_writes(f.read())
            if found:
                raise RuntimeError(f"{tmp}/{name}: vector instructions behind an empty execution mask: "
                                   + "; ".join(found[:5]))
    os.replace(os.path.join(tmp, "out.o"), obj)
    shutil.rmtree(tmp)
    return r


def build(verbose: bool = False, jobs: int | None = None) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(8, os.cpu_count() or 1)
    src_k = os.path.join(CSRC, "sq_kernels.hip")
    src_t = os.path.join(CSRC, "sq_tile_kernels.hip")
    parts = [(g, 0) for g in CUBE_GROUPS] + [(g, 1) for g in TWO_ROW_GROUPS]
    work = []  # (command, object)
    for i, (group, two) in enumerate(parts):
        cubes = " ".join(f"X({c})" for c in group)
        defs = [f"-DSQ_CUBES={cubes}", "-DSQ_PART=%d" % i, "-DSQ_TWO_ROWS=%d" % two]
        work.append(([HIPCC, *DEVICE_FLAGS, *defs, src_k], f"sq_kernels_{i}.o"))
    for c in reversed(TILE_CUBES):
        work.append(([HIPCC, *DEVICE_FLAGS, *TILE_FLAGS, f"-DSQ_CUBES=X({c})", src_t], f"sq_tile_{c}.o"))
    work.append(([HIPCC, *DEVICE_FLAGS, "-DSQ_COMMON_ONLY", src_k], "sq_common.o"))
    work.append(([CXX, *HOST_FLAGS, os.path.join(CSRC, "sq_api.cpp")], "sq_api.o"))
    objs = [os.path.join(BUILD, name) for _, name in work]
    with ThreadPoolExecutor(jobs) as ex:
        for r in ex.map(_compile, [cmd for cmd, _ in work], objs):
            if verbose and r.stderr:
                sys.stderr.write(r.stderr)
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
