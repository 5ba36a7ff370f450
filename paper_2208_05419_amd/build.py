"""Build the HIP library (gfx950) in-tree: paper_2208_05419_amd/libafno_mi355x.so."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libafno_mi355x.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 vector ops stay off (hipcc -O3 would otherwise form them from float2 code)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


# (source, its own flags): compiled side by side, then linked.  afno_kernels.hip and
# afno_api.cpp alone make the same library (afno_rows.hip is then part of the first).
UNITS = [(os.path.join(CSRC, "afno_kernels.hip"), ["-DAFNO_SEPARATE_ROWS"])] + [
    (os.path.join(CSRC, "afno_rows.hip"), [f"-DAFNO_ROWS_PART={p}"]) for p in range(4)
] + [(os.path.join(CSRC, "afno_api.cpp"), [])]


def build(verbose: bool = False, extra=()) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f"{i}.o") for i in range(len(UNITS))]

        def compile_one(unit, obj):
            cmd = [HIPCC, *FLAGS, "-c", *extra, *unit[1], "-x", "hip", unit[0], "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)

        with ThreadPoolExecutor(max_workers=min(len(UNITS), os.cpu_count() or 1)) as pool:
            for f in [pool.submit(compile_one, u, o) for u, o in zip(UNITS, objs)]:
                f.result()
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB + ".tmp"],
                       check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
