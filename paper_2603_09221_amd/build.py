"""Build of the HIP library for gfx950: every kernel family is its own translation unit (and, where the
kernels are templates over the state size, one object per state size), compiled in parallel and linked
into paper_2603_09221_amd/lib/libttc_lqr.so.

    python -m paper_2603_09221_amd.build [--force] [-j N]

Without --force only objects older than a source file are rebuilt.
"""
from __future__ import annotations

import argparse
import glob
import os
import re
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG), "include")
OBJDIR = os.path.join(PKG, "lib", "_build")
OUT = os.path.join(PKG, "lib", "libttc_lqr.so")

HIPCC_FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# (source, state sizes it is compiled for; None = once)
UNITS = [("ttc_api.hip", None),
         ("k_solve.hip", (32, 64, 128)),
         ("k_doubling.hip", (16, 32, 64, 128)),
         ("k_squaring.hip", (32, 64, 128)),
         ("k_rollout.hip", (16, 32, 64, 128)),
         ("k_tv.hip", (16, 32, 64, 128)),
         ("k_scan.hip", (16, 32, 64, 128)),
         ("k_backward.hip", (16, 32, 64, 128)),
         ("k_small.hip", None),
         ("k_squaring16.hip", None),
         ("k_tv_small.hip", None),
         ("k_cxt.hip", None),
         ("k_cxt_bwd.hip", None),
         ("k_block.hip", None)]

# Per (source, state size) compile flags: wavefronts of one 16-wide block each (twice as many per problem) instead of
# two, where measured faster.  The Riccati and squaring kernels own matrices by columns: at d = 64 one column tile a wavefront
# leaves room for three workgroups a compute unit.  The sequential product is faster with fewer, fatter wavefronts (its constant
# operands stay in registers; at d = 64 four problems fit a compute unit).  Measured with one block against two: squaring path
# d = 128, T = 16, 8192 problems 11.6 ms against 14.9, d = 64, T = 8, 16384 problems 2.55 against 2.73; with products in float32,
# roll-out d = 128, T = 8, 1024 problems 2.75 ms against 3.04; flagged doubling d = 128, T = 16 501k problems/s against 488k.
_ONE_ROW_BLOCK = "-DTTC_ROW_BLOCKS(D)=((D)==%d?1:((D)>=32?2:1))"
# The backward kernel at d = 64 takes more registers by itself; held to the 168 of three wavefronts a SIMD it spills 14 of them (7 with
# bfloat16 inputs) and is still the faster (T = 8, 8192 problems, time-invariant 2.26 ms against 2.88).  At d = 128 two column tiles a
# wavefront leave one wavefront a SIMD, which waits for what it spills (512 problems 1.35 ms against 1.05).
_THREE_WAVES = "-DTTC_COLS_WAVES(D)=3"
UNIT_FLAGS = {("k_backward.hip", 64): [_ONE_ROW_BLOCK % 64, _THREE_WAVES],
              ("k_backward.hip", 128): [_ONE_ROW_BLOCK % 128],
              ("k_tv.hip", 64): [_ONE_ROW_BLOCK % 64],
              ("k_tv.hip", 128): [_ONE_ROW_BLOCK % 128],
              ("k_doubling.hip", 128): [_ONE_ROW_BLOCK % 128],
              ("k_rollout.hip", 64): [_ONE_ROW_BLOCK % 64],
              ("k_rollout.hip", 128): [_ONE_ROW_BLOCK % 128],
              ("k_squaring.hip", 64): [_ONE_ROW_BLOCK % 64],
              ("k_squaring.hip", 128): [_ONE_ROW_BLOCK % 128]}

# Sources whose functions that are not inlined read and write the problems' matrices (not one by one, as those of the split products)
NO_FLAT = ("k_squaring16.hip",)

# Vector registers that a kernel of a unit may spill: these lose time by what is inlined into them (the inverse of a pivot block, the recursion)
MOST_SPILLED = {("k_solve.hip", 128): 160, ("k_tv.hip", 128): 90}

_NOISE = "is not a recognized feature for this target"


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if _NOISE not in l and "warning generated" not in l)
    if res.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), err))
    if err.strip():
        print(err, file=sys.stderr)


def misplaced_vector_moves(asm: str) -> list:
    """(kernel, line number, instruction) of vector spills, reloads and copies that stand between the label a wavefront
    with no active lane jumps to (s_cbranch_execz) and the instruction there that restores EXEC.

    The compiler this was built with places them so now and then, when it spills scalar registers at the same join: a
    wavefront that skipped the branch then runs them with EXEC = 0 and keeps a stale register or scratch slot (a wrong
    info, or a wild address and a memory fault).  What provokes it is a branch taken by masking lanes off, on a condition
    that is the same for a whole wavefront, under high register pressure; the cure is to make that branch scalar (see
    uniform() in ttc_device.hpp)."""
    skipped_to = set(re.findall(r"^\s+s_cbranch_execz\s+(\S+)", asm, re.M))
    kernel, pending, found = None, None, []
    for n, line in enumerate(asm.split("\n"), 1):
        label = re.match(r"^([\w.$]+):", line)
        if label:
            if label.group(1).startswith(".LBB"):
                pending = [] if label.group(1) in skipped_to else None
            elif not label.group(1).startswith("."):
                kernel, pending = label.group(1), None
        elif pending is None:
            continue
        elif re.match(r"\s+s_(or|mov)_b64 exec,", line):
            found += pending
            pending = None
        elif re.match(r"\s+(scratch_|buffer_|v_accvgpr_|v_mov_b)", line):
            pending.append((kernel, n, line.strip()))
        elif re.match(r"\s+s_(cbranch|branch|endpgm|barrier|\w+ exec|\w*saveexec)", line) or \
                not re.match(r"\s*(;|s_|v_readlane|v_writelane|$)", line):
            pending = None  # the join's own code has begun
    return found


def flat_accesses(asm: str) -> list:
    """(kernel or function, line number, instruction) of flat memory instructions: reads and writes through a pointer of which the
    compiler could not see whether it is to device memory or to LDS.  The counters of both wait for them; in_memory() and in_lds()
    in ttc_device.hpp tell a function that is not inlined."""
    function, found = None, []
    for n, line in enumerate(asm.split("\n"), 1):
        label = re.match(r"^([A-Za-z_$][\w$]*):", line)
        if label:
            function = label.group(1)
        elif re.match(r"\s+flat_(load|store|atomic)", line):
            found.append((function, n, line.strip()))
    return found


def spilled_registers(asm: str) -> list:
    """(kernel, vector registers spilled) of a listing, from the kernels' metadata at its end."""
    return [(name, int(count)) for name, count in
            re.findall(r"^\s+\.name:\s+(_Z\w+)$(?:(?!^\s+\.name:).)*?^\s+\.vgpr_spill_count:\s+(\d+)$", asm, re.M | re.S)]


def _compile(job):
    """Compile one object in a folder of its own, where the compiler leaves its assembly, and look through that."""
    cmd, obj = job
    folder = obj[:-2]
    shutil.rmtree(folder, ignore_errors=True)
    os.makedirs(folder)
    out = os.path.join(folder, os.path.basename(obj))
    _run(cmd + ["-save-temps=obj", "-o", out])
    listings = glob.glob(os.path.join(folder, "*gfx950.s"))
    if len(listings) != 1:
        raise RuntimeError("%s: %d device listings" % (out, len(listings)))
    with open(listings[0]) as f:
        asm = f.read()
    unit = (os.path.basename(cmd[-1]), next((int(a[8:]) for a in cmd if a.startswith("-DTTC_D=")), None))
    spilled = [x for x in spilled_registers(asm) if x[1] > MOST_SPILLED.get(unit, x[1])]
    if spilled:
        raise RuntimeError("more than %d spilled vector registers (%s): %s" % (MOST_SPILLED[unit], " ".join(cmd), spilled))
    for what, found in (("vector instructions ahead of an EXEC restore", misplaced_vector_moves(asm)),
                        ("flat memory instructions", flat_accesses(asm) if unit[0] in NO_FLAT else [])):
        if found:
            raise RuntimeError("%s (%s):\n%s" % (what, " ".join(cmd), "\n".join("%s line %d: %s" % x for x in found)))
    os.replace(out, obj)
    shutil.rmtree(folder)


def _newest_source():
    t = 0.0
    for folder in (CSRC, INCLUDE):
        for name in os.listdir(folder):
            t = max(t, os.path.getmtime(os.path.join(folder, name)))
    return max(t, os.path.getmtime(os.path.abspath(__file__)))


def build(force: bool = True, jobs: int | None = None, extra_flags=()) -> str:
    """Compile and link; returns the path of the shared library."""
    os.makedirs(OBJDIR, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = jobs or min(16, os.cpu_count() or 1)
    newest = _newest_source()
    work, objs = [], []
    for src, sizes in UNITS:
        for d in (sizes or (None,)):
            stem = os.path.splitext(src)[0] + ("" if d is None else "_%d" % d)
            obj = os.path.join(OBJDIR, stem + ".o")
            objs.append(obj)
            if force or not os.path.exists(obj) or os.path.getmtime(obj) < newest:
                cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + UNIT_FLAGS.get((src, d), []) + \
                      (["-DTTC_D=%d" % d] if d else []) + ["-c", os.path.join(CSRC, src)]
                work.append((cmd, obj))
    # the largest state sizes take longest: start them first
    work.sort(key=lambda c: -max([int(a[8:]) for a in c[0] if a.startswith("-DTTC_D=")] or [0]))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        list(ex.map(_compile, work))
    if work or not os.path.exists(OUT):
        _run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", OUT] + objs)
    return OUT


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--force", action="store_true")
    ap.add_argument("-j", type=int, default=None)
    ap.add_argument("--flag", action="append", default=[], help="extra hipcc flag (repeatable), e.g. --flag=-DTTC_PHASE_TIMERS")
    a = ap.parse_args()
    print(build(force=a.force, jobs=a.j, extra_flags=a.flag))
