"""Build libelb.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

Usage: python -m paper_2211_16933_amd.build   (or call build()).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libelb.so")
SOURCES = ["elb.hip", "host_math.cpp", "stage_kernels.hip"]
HEADERS = ["closure_kernels.h", "elb_kernels.h", "host_math.h", "mlp_device.h", "node_tables.h",
           "readout_kernels.h", "stage_table.h", "state_kernels.h"]
# stage_kernels.hip is compiled once per mode of the stage kernel
STAGE_MODES = {"f64": 0, "f32": 1, "mixed": 2, "fixup": 3}

FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         # packed FP32 instructions are kept out of every kernel on this target
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _run(cmds, verbose):
    """Run the commands side by side; raise with the output of the first that fails."""
    procs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    outs = [p.communicate()[0] for p in procs]
    for p, out in zip(procs, outs):
        if p.returncode != 0:
            sys.stderr.write(out)
            raise RuntimeError("hipcc failed building libelb.so")


def build(verbose: bool = False) -> str:
    objdir = os.path.join(HERE, "build")
    os.makedirs(objdir, exist_ok=True)
    objs, cmds = [], []
    jobs = [("stage_kernels.hip", f"stage_{m}.o", [f"-DELB_STAGE_MODE={v}"]) for m, v in STAGE_MODES.items()]
    jobs += [("elb.hip", "elb.o", []), ("host_math.cpp", "host_math.o", [])]
    for src, obj, extra in jobs:
        objs.append(os.path.join(objdir, obj))
        cmds.append(["hipcc", *FLAGS, *extra, "-c", "-o", objs[-1], os.path.join(CSRC, src)])
    _run(cmds, verbose)
    tmp = LIB + ".tmp"
    _run([["hipcc", "--offload-arch=gfx950", "-shared", "-o", tmp, *objs]], verbose)
    os.replace(tmp, LIB)
    return LIB


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    files = SOURCES + HEADERS
    paths = [os.path.join(CSRC, f) for f in files] + [os.path.join(os.path.dirname(HERE), "include", "elb.h")]
    return any(os.path.getmtime(p) > t for p in paths)


if __name__ == "__main__":
    print(build(verbose=True))
