"""Builds librnnt_beam.so for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librnnt_beam.so")
# (source, defines): compiled at the same time, then linked
UNITS = [("rnnt_beam.hip", []), ("rnnt_lm.hip", []), ("rnnt_resident.hip", [])] + [
    ("resident_kernels.hip", [f"-DRB_RES_FULL={full}", f"-DRB_RES_FORM={form}", f"-DRB_RES_ST={st}"])
    for st in (0, 1) for full in (1, 0) for form in (0, 1, 2)]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-Wno-unused-value",
         "-Wno-pass-failed", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd: list, verbose: bool) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err)


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f"{i}.o") for i in range(len(UNITS))]
        cmds = [[HIPCC] + FLAGS + defs + ["-c", "-o", o, os.path.join(CSRC, src)] for (src, defs), o in zip(UNITS, objs)]
        with ThreadPoolExecutor(max_workers=min(8, int(os.environ.get("MAX_JOBS", "8")))) as pool:
            list(pool.map(lambda c: _run(c, verbose), cmds))
        _run([HIPCC] + FLAGS + ["-shared", "-o", LIB] + objs, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
