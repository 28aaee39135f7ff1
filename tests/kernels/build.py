"""Builds tests/kernels/libtest_kernels.so for gfx950: device functions of the
library, called by test kernels of their own."""
import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
LIB = os.path.join(HERE, "libtest_kernels.so")
# source -> options of its own
SOURCES = {"tile_cache.hip": ["-DRF_TRACK_BLOCK=512"], "reciprocals.hip": []}


def build() -> str:
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    from paper_1905_02082_amd import build as hip
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("%s failed:\n%s\n%s" % (" ".join(cmd), r.stdout, r.stderr))

    def compile_one(src):
        obj = os.path.join(objdir, src + ".o")
        run([hip.HIPCC, *hip.FLAGS, "-fvisibility=hidden", *SOURCES[src], "-c", os.path.join(HERE, src), "-o", obj])
        return obj

    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    run([hip.HIPCC, "--offload-arch=" + hip.ARCH, "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
