"""Build libtip.so (HIP, gfx950) in-tree.

    python -m paper_1302_4018_amd.build [--resource-usage]

Compiles every source under csrc/ with hipcc for gfx950 only and links one
shared library next to this file.  Packed FP32 instructions are disabled for
all device code (-packed-fp32-ops).
"""

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libtip.so")
SOURCES = ["tip_kernels.hip", "tip_api.hip", "tip_bandwidth.hip", "tip_batch.hip", "tip_resident.hip", "tip_resident_cov.hip",
           "tip_resident_2d.hip", "tip_resident_3d.hip", "tip_resident_4d.hip", "tip_cluster.hip",
           "tip_cluster_2d.hip", "tip_cluster_3d.hip", "tip_cluster_4d.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src, extra):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    return src, obj, r


def build(resource_usage=False, verbose=True):
    os.makedirs(BUILD, exist_ok=True)
    extra = ["-Rpass-analysis=kernel-resource-usage"] if resource_usage else []
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        results = list(ex.map(lambda s: _compile(s, extra), SOURCES))
    objs = []
    for src, obj, r in results:
        if verbose and (r.stderr.strip() and (resource_usage or r.returncode != 0)):
            sys.stderr.write(r.stderr)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr[-4000:]}")
        objs.append(obj)
    tmp = LIB + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-4000:]}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(resource_usage="--resource-usage" in sys.argv))
