"""Build the gfx950 HIP library ``libzmc.so`` in-tree.

    python -m paper_1902_07916_amd.build [--jobs N]

Compiles the sampling kernel once per integrand (-DZMC_F=<id>), the level
kernels, the engine and the C ABI with hipcc for gfx950, in parallel, and
links them into ``paper_1902_07916_amd/libzmc.so``.
"""
from __future__ import annotations

import argparse
import json
import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libzmc.so")
N_INTEGRANDS = 8

HIP_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    "-I" + INCLUDE, "-I" + CSRC,
    # no packed FP32 instructions (v_pk_*_f32) anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]

# The sampling kernels' own flags.  Loop headers on 64-byte lines: the
# sampling loop's speed moved by up to 6% with where its header fell in a
# line.  Scheduling for the fewest registers: each Philox block's chain then
# runs depth first, dependent instructions one after another, instead of all
# blocks round by round.  One wave issues a vector instruction every 4-5
# cycles at best either way (measured), so a chain's latency costs nothing
# beside other waves.  Same source, points/s: 6-D sine FP32 5.40e11 -> 5.75e11,
# 6-D Genz Gaussian 5.25e11 -> 5.60e11, 12-D corner peak 2.77e11 -> 2.86e11;
# VGPRs at 6, 9 and 12-D: 73 -> 60, 132 -> 96, 134 -> 104.
SAMPLE_FLAGS = ["-falign-loops=64", "-mllvm", "-amdgpu-sched-strategy=iterative-minreg"]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


RTC_HEADERS = (("zmc.h", os.path.join(INCLUDE, "zmc.h")),
               ("zmc_device.hpp", os.path.join(CSRC, "zmc_device.hpp")),
               ("zmc_trig.hpp", os.path.join(CSRC, "zmc_trig.hpp")),
               ("zmc_sample_core.hpp", os.path.join(CSRC, "zmc_sample_core.hpp")))
RTC_STUBS = (("hip/hip_runtime.h", "// built into hipRTC\n"),
             ("stdint.h", "// integer types come from the hipRTC prelude\n"))


def write_rtc_embed() -> str:
    """Embed the device headers the run-time compiled kernels include, as
    string literals (zmc_rtc_embed.inc in the build directory)."""
    path = os.path.join(BUILD, "zmc_rtc_embed.inc")
    names, srcs = [], []
    for name, f in RTC_HEADERS:
        with open(f) as fh:
            text = fh.read()
        if ")ZMCRTC\"" in text:
            raise RuntimeError("delimiter clash in " + f)
        names.append(name)
        srcs.append(text)
    for name, text in RTC_STUBS:
        names.append(name)
        srcs.append(text)
    out = ["// generated by paper_1902_07916_amd/build.py: device headers for hipRTC"]
    out.append("static const int kRtcHeaderCount = %d;" % len(names))
    out.append("static const char* kRtcHeaderNames[] = {%s};" % ", ".join('"%s"' % n for n in names))
    out.append("static const char* kRtcHeaderSources[] = {")
    for t in srcs:
        out.append('R"ZMCRTC(' + t + ')ZMCRTC",')
    out.append("};")
    text = "\n".join(out) + "\n"
    old = open(path).read() if os.path.exists(path) else None
    if old != text:
        with open(path, "w") as fh:
            fh.write(text)
    return path


def _units():
    units = []
    for f in range(N_INTEGRANDS):
        units.append((os.path.join(CSRC, "zmc_sample.hip"), os.path.join(BUILD, f"zmc_sample_{f}.o"),
                      [f"-DZMC_F={f}"] + SAMPLE_FLAGS))
    # the per-cube / per-integral kernels round every product and sum
    # separately, in the order the method states them (no FMA contraction)
    units.append((os.path.join(CSRC, "zmc_level.hip"), os.path.join(BUILD, "zmc_level.o"), ["-ffp-contract=off"]))
    units.append((os.path.join(CSRC, "zmc_engine.hip"), os.path.join(BUILD, "zmc_engine.o"), ["-I" + BUILD]))
    units.append((os.path.join(CSRC, "zmc_abi.hip"), os.path.join(BUILD, "zmc_abi.o"), []))
    units.append((os.path.join(CSRC, "zmc_rtc.hip"), os.path.join(BUILD, "zmc_rtc.o"), ["-I" + BUILD]))
    return units


def _deps_mtime() -> float:
    """Newest of the files every translation unit may depend on."""
    files = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hpp", ".json"))]
    files += [os.path.join(INCLUDE, "zmc.h"), os.path.abspath(__file__)]
    files += [os.path.join(BUILD, f) for f in os.listdir(BUILD) if f.endswith(".inc")]
    return max(os.path.getmtime(f) for f in files)


def _compile(src, obj, extra, skip_if_newer=None):
    if skip_if_newer is not None and os.path.exists(obj) and \
            os.path.getmtime(obj) > max(skip_if_newer, os.path.getmtime(src)):
        return obj
    cmd = [hipcc()] + HIP_FLAGS + extra + ["-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s%s" % (" ".join(cmd), res.stdout, res.stderr))
    return obj


TUNE_DEFAULT = os.path.join(CSRC, "zmc_tune_gfx950.json")
WAVE_HINTS = (1, 4, 5, 6)  # must match kWaveHints in zmc_kernels.hpp


def write_tune_default() -> str:
    """_build/zmc_tune_default.inc: the built-in occupancy variant and block
    shape per (integrand, dim, eval), from the measured table
    zmc_tune_gfx950.json (keys "integrand:dim:eval:w" -> waves per
    SIMD, absent = 1; "integrand:dim:eval:b" -> threads per block, absent =
    256)."""
    table = json.load(open(TUNE_DEFAULT)) if os.path.exists(TUNE_DEFAULT) else {}
    idx = [[[0, 0] for _ in range(17)] for _ in range(N_INTEGRANDS)]
    for key, w in table.items():
        parts = key.split(":")
        if len(parts) == 4 and parts[3] == "w" and int(w) in WAVE_HINTS:
            f, d, e = int(parts[0]), int(parts[1]), int(parts[2])
            if 0 <= f < N_INTEGRANDS and 1 <= d <= 16 and e in (0, 1):
                idx[f][d][e] = WAVE_HINTS.index(int(w))
    blk = [[[256, 256] for _ in range(17)] for _ in range(N_INTEGRANDS)]
    for key, b in table.items():
        parts = key.split(":")
        if len(parts) == 4 and parts[3] == "b" and int(b) in (64, 128, 256):
            f, d, e = int(parts[0]), int(parts[1]), int(parts[2])
            if 0 <= f < N_INTEGRANDS and 1 <= d <= 16 and e in (0, 1):
                blk[f][d][e] = int(b)
    rows = ",\n".join("    {" + ", ".join("{%d, %d}" % (a, b) for a, b in idx[f]) + "}" for f in range(N_INTEGRANDS))
    brows = ",\n".join("    {" + ", ".join("{%d, %d}" % (a, b) for a, b in blk[f]) + "}" for f in range(N_INTEGRANDS))
    out = os.path.join(BUILD, "zmc_tune_default.inc")
    text = ("// generated by build.py from zmc_tune_gfx950.json\n"
            "static const unsigned char kDefaultWaveHint[%d][17][2] = {\n%s};\n"
            "static const short kDefaultBlock[%d][17][2] = {\n%s};\n" % (N_INTEGRANDS, rows, N_INTEGRANDS, brows))
    if not os.path.exists(out) or open(out).read() != text:
        with open(out, "w") as fh:
            fh.write(text)
    return out


def build(jobs: int | None = None, verbose: bool = False, incremental: bool = False) -> str:
    """Compile every translation unit and link libzmc.so; returns its path.
    incremental: keep objects newer than their source and every header."""
    os.makedirs(BUILD, exist_ok=True)
    write_rtc_embed()
    write_tune_default()
    jobs = jobs or min(8, os.cpu_count() or 4)
    units = _units()
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        newest = _deps_mtime() if incremental else None
        futs = [ex.submit(_compile, *u, skip_if_newer=newest) for u in units]
        objs = [f.result() for f in futs]
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + ["-lhiprtc", "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed: %s\n%s%s" % (" ".join(cmd), res.stdout, res.stderr))
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


def main(argv=None) -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=None)
    ap.add_argument("--incremental", action="store_true",
                    help="keep objects that are newer than their source and every header")
    a = ap.parse_args(argv)
    build(a.jobs, verbose=True, incremental=a.incremental)
    return 0


if __name__ == "__main__":
    sys.exit(main())
