"""Build libamgiga.so in the package directory (gfx950 only).

Host setup code is compiled by g++ without FMA contraction (its bits define
the aggregates); the HIP sources by hipcc for gfx950 with packed-FP32
instructions disabled, one process per source.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libamgiga.so")
HIP_SOURCES = ["solver.hip", "blk_win.hip", "blk_wins.hip", "blk_rows.hip", "blk_post.hip", "split.hip",
               "probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _run(cmd):
    subprocess.check_call(cmd)


def build(verbose=False):
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    hip = [HIPCC, "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-result"]
    jobs = {"host_setup.cpp": ["g++", "-O2", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math", "-pthread",
                               "-Wall"],
            # device set-up: no FMA contraction (its bits must equal the host set-up's)
            "setup_dev.hip": hip + ["-ffp-contract=off"]}
    jobs.update({src: hip for src in HIP_SOURCES})
    objs = [os.path.join(bdir, src.rsplit(".", 1)[0] + ".o") for src in jobs]
    cmds = [cmd + inc + ["-c", os.path.join(CSRC, src), "-o", obj] for (src, cmd), obj in zip(jobs.items(), objs)]
    with ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 1)) as pool:
        list(pool.map(_run, cmds))
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs, "-pthread",
          "-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx"])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
