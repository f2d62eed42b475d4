"""The host runtime (everything but the kernels) built against a stand-in for the
HIP runtime, so that its order of calls, its error paths and its bookkeeping run
and can be watched on a CPU.  ``load()`` returns the Python binding on that
library, with ``stub`` (the stand-in's own entry points) and ``Watch``."""
import ctypes
import importlib.util
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(os.path.dirname(HERE)), "paper_2609_09322_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC"]
HOOK = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_char_p, ctypes.c_void_p, ctypes.c_void_p)


def build(out_dir):
    sources = [os.path.join(PKG, "csrc", f"dart_{n}.hip")
               for n in ("runtime", "server", "stream", "noalloc")]
    sources.append(os.path.join(HERE, "hip_stub.cpp"))

    def compile_one(src):
        obj = os.path.join(out_dir, os.path.basename(src) + ".o")
        subprocess.check_call([HIPCC, "-x", "hip"] + FLAGS + ["-c", src, "-o", obj])
        return obj

    with ThreadPoolExecutor(max_workers=5) as ex:
        objs = list(ex.map(compile_one, sources))
    # (host objects name the device code that is not there)
    names = subprocess.run(["nm", "-u"] + objs, capture_output=True, text=True, check=True).stdout
    absent = sorted({w for w in names.split() if w.startswith("__hip_fatbin")})
    lib = os.path.join(out_dir, "libdart_host.so")
    subprocess.check_call(["g++", "-shared", "-o", lib] + objs + ["-Wl,-Bsymbolic", "-lpthread"] +
                          [f"-Wl,--defsym={w}=0" for w in absent])
    return lib


def load():
    with tempfile.TemporaryDirectory() as d:
        lib = build(d)
        spec = importlib.util.spec_from_file_location("dart_on_stub", os.path.join(PKG, "dart.py"))
        dart = importlib.util.module_from_spec(spec)
        sys.modules[spec.name] = dart  # (dataclasses look their module up)
        spec.loader.exec_module(dart)
        dart.LIB_PATH = lib
        stub = dart._load()
    for name, res, args in (("stub_hook", None, [HOOK]), ("stub_room", None, [ctypes.c_size_t]),
                            ("stub_bad_element", None, [ctypes.c_uint64]),
                            ("stub_hold_host_funcs", None, [ctypes.c_int]),
                            ("stub_run_host_funcs", None, []),
                            ("stub_event_alive", ctypes.c_int, [ctypes.c_void_p]),
                            ("stub_held", ctypes.c_size_t, [])):
        f = getattr(stub, name)
        f.restype, f.argtypes = res, args
    dart.stub = stub
    return dart


class Watch:
    """Calls made while the block runs, as (name, a, b); `answer(name, a, b)` may
    return the error a call is to give instead of being run."""

    def __init__(self, dart, answer=None):
        self.dart, self.answer, self.calls = dart, answer, []

        def hook(name, a, b):
            n = name.decode()
            self.calls.append((n, a, b))
            return (self.answer(n, a, b) or 0) if self.answer else 0

        self._hook = HOOK(hook)

    def __enter__(self):
        self.dart.stub.stub_hook(self._hook)
        return self

    def __exit__(self, *exc):
        self.dart.stub.stub_hook(ctypes.cast(None, HOOK))

    def names(self):
        return [c[0] for c in self.calls]

    def of(self, name):
        return [c for c in self.calls if c[0] == name]
