"""Builds liblqfire.so (hipcc, gfx950) in-tree."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INC = os.path.join(ROOT, "include")
BUILD = os.environ.get("LQ_BUILD_DIR", os.path.join(HERE, "_build"))
LIB = os.environ.get("LQ_LIB_OUT", os.path.join(HERE, "liblqfire.so"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-I", INC, "-I", CSRC] + os.environ.get("LQ_EXTRA_FLAGS", "").split()
# packed FP32 instructions stay off for all device code
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-ffp-contract=on"]
SOURCES = [
    ("march_f64.hip", DEVICE),
    ("march_f32.hip", DEVICE),
    ("kernels.hip", DEVICE),
    ("brick.hip", DEVICE),
    ("observe.hip", DEVICE),
    ("noalloc.hip", DEVICE),
    ("stream_copy.hip", DEVICE),
    ("abi.cpp", []),
    ("geometry.cpp", ["-ffp-contract=off"]),
]


def _compile(src, extra):
    obj = os.path.join(BUILD, src + ".o")
    cmd = [HIPCC] + COMMON + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build() -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(lambda s: _compile(*s), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
