"""Build libnsc.so in-tree with hipcc for gfx950 (no JIT cache)."""
import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libnsc.so")
SOURCES = ["nsc_host.cpp", "k_nonlinear.hip", "k_solve.hip", "k_stage.hip", "k_restart.hip",
           "k_diag.hip", "k_noalloc.hip"] + ["k_len%d.hip" % i for i in range(1, 13)]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed FP32 instructions are kept out of generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    return res.stderr


def build(verbose=False):
    tmp = OUT + ".tmp"
    objs = tempfile.mkdtemp(prefix="nsc_build_")
    try:
        # one object per source, several at a time
        jobs = [["hipcc"] + FLAGS + ["-c", os.path.join(CSRC, s), "-o", os.path.join(objs, s + ".o")]
                for s in SOURCES]
        workers = min(len(jobs), len(os.sched_getaffinity(0)), 8)
        with ThreadPoolExecutor(workers) as pool:
            logs = list(pool.map(_run, jobs))
        logs.append(_run(["hipcc"] + FLAGS + ["-shared", "-o", tmp] + [j[-1] for j in jobs]))
    finally:
        shutil.rmtree(objs, ignore_errors=True)
    if verbose:
        print("".join(logs))
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
