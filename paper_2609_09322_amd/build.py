"""Builds the HIP library ``libdart.so`` for gfx950 (in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libdart.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = ["dart_kernels.hip", "dart_runtime.hip", "dart_server.hip", "dart_stream.hip",
           "dart_noalloc.hip"]
# The march kernels are compiled once per (storage type, ray precision), in
# parallel: hundreds of instances in one unit took five minutes.
MARCH_UNITS = [("f64", 0, 1), ("f32", 1, 1), ("f16", 2, 0), ("f16_r64", 2, 1), ("bf16", 3, 0),
               ("bf16_r64", 3, 1)]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Wno-unused-result",
         # no packed FP32 instructions anywhere in the device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build(out: str = OUT, defines=()) -> str:
    obj_dir = os.path.join(HERE, "_build" + ("_" + "_".join(d.replace("=", "") for d in defines) if defines else ""))
    os.makedirs(obj_dir, exist_ok=True)

    units = [("dart_kernels.hip", "dart_march_%s.o" % name,
              ["DART_MARCH_STORE=%d" % store, "DART_MARCH_F64_RAYS=%d" % f64])
             for name, store, f64 in MARCH_UNITS]
    units += [(src, src.replace(".hip", ".o"), []) for src in SOURCES]

    def compile_one(unit):
        src, name, extra = unit
        obj = os.path.join(obj_dir, name)
        subprocess.check_call([HIPCC] + FLAGS + ["-D" + d for d in list(defines) + extra]
                              + ["-c", os.path.join(CSRC, src), "-o", obj])
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_one, units))
    tmp = out + ".tmp"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
                          + ["-lpthread"])
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build())
