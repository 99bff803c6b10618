"""Builds libchunkflow.so (host planner + HIP kernels for gfx950) in-tree with hipcc."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libchunkflow.so")
HOST_SOURCES = ["planner.cpp"]
HIP_SOURCES = ["api.hip", "attn_simple.hip", "attn_fp32.hip", "attn_mfma_fwd.hip", "attn_mfma_bwd.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed-fp32 VALU forms are switched off for all device code.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
             "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
RESOURCE_REPORT = "-Rpass-analysis=kernel-resource-usage"


def _stale(obj, deps):
    return not os.path.exists(obj) or any(os.path.getmtime(d) > os.path.getmtime(obj) for d in deps)


def _resources(report):
    """(kernel, name, value) of a compiler resource report."""
    kernel = None
    for line in report.splitlines():
        m = re.search(r"remark: [^:]*?(Function Name|VGPRs Spill|ScratchSize \[bytes/lane\]): (\S+)", line)
        if m is None:
            continue
        if m[1] == "Function Name":
            kernel = m[2]
        else:
            yield kernel, m[1], int(m[2])


def spilled_accumulators(report):
    """Kernels of a compiler resource report that update accumulators in place behind the compiler's back (the dK/dV kernels
    at head_dim 128; mfma_common.h, accumulate_in_place) and spill: a spilled accumulator would be stored while its last
    MFMA is still running.  -> [(kernel, what)]"""
    return [(k, f"{what}: {n}") for k, what, n in _resources(report) if "mfma_dkv" in k and "ILi128E" in k and n != 0]


def spilled_operands(report):
    """Matrix kernels that spill vector registers: their blocks are laid out to fit, and a few reloads in the loop over blocks
    take what the layout gained (fp32 step of 3 packed chunks of 532 tokens, 4 heads, D = 128: 79 us with 26 spilled in the
    backward, 71 with none).  -> [(kernel, what)]"""
    return [(k, f"{what}: {n}") for k, what, n in _resources(report)
            if what == "VGPRs Spill" and n != 0 and re.search(r"\d(mfma|f32)_\w+_kernel", k)]


def build(force=True, verbose=False):
    """Compile every source and link the shared library.  force=False rebuilds only stale objects."""
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    headers = [os.path.join(ROOT, "include", "chunkflow.h")] + \
              [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    objs, procs = [], []
    for src in HOST_SOURCES + HIP_SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(bdir, src + ".o")
        objs.append(obj)
        if not force and not _stale(obj, [path] + headers):
            continue
        if src.endswith(".hip"):
            cmd = [HIPCC] + HIP_FLAGS + [RESOURCE_REPORT, "-fno-caret-diagnostics"] + inc + ["-c", path, "-o", obj]
        else:
            cmd = [HIPCC, "-O2", "-std=c++17", "-fPIC", "-Wall", "-Wextra"] + inc + ["-x", "c++", "-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = []
    for src, pr in procs:
        out, _ = pr.communicate()
        spilled, slow = spilled_accumulators(out), spilled_operands(out)
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and RESOURCE_REPORT not in l)
        if pr.returncode != 0:
            failed.append(f"--- {src}\n{out}")
        elif spilled:
            os.remove(os.path.join(bdir, src + ".o"))
            failed.append(f"--- {src}: kernels with in-place accumulators may not spill: {spilled}")
        elif slow:
            os.remove(os.path.join(bdir, src + ".o"))
            failed.append(f"--- {src}: matrix kernels may not spill: {slow}")
        elif verbose and out.strip():
            print(out)
    if failed:
        raise RuntimeError("hipcc failed:\n" + "\n".join(failed))
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(force="--force" in sys.argv, verbose=True))
