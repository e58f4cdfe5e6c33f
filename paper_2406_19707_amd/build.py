"""Builds libinfinigen_hip.so for gfx950 with hipcc (cross-compiles without a GPU)."""
from __future__ import annotations

import importlib.util
import os
import runpy
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libinfinigen_hip.so")
CALL = os.path.join(HERE, "_ig_call" + sysconfig.get_config_var("EXT_SUFFIX"))    # for this Python alone
SOURCES = ["ig_api.hip", "k_scan.hip", "k_project.hip", "k_kv.hip", "k_layer.hip", "k_equalize.hip", "k_index.hip", "k_skew.hip", "ig_host.cpp"]
HIPCC = "/opt/rocm/bin/hipcc"
# packed-fp32 instruction selection is switched off for every device compile
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if src.endswith(".hip"):
        cmd = [HIPCC, *COMMON, *DEVICE_FLAGS, "-c", path, "-o", obj]
    else:
        cmd = [HIPCC, *COMMON, "-x", "c++", "-c", path, "-o", obj]
    subprocess.check_call(cmd)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.check_call([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs])
    _build_call()
    if verbose:
        print("built", LIB)
    return LIB


def _build_call() -> None:
    """The marshalling module of the Python binding: host code over the library and torch's tensor class.  It only makes
    calls cheaper, so without torch, its headers or Python's the build goes on without it (and without an old one, which
    may be of another library): the binding marshals through ctypes then."""
    if os.path.exists(CALL):
        os.remove(CALL)
    spec = importlib.util.find_spec("torch")
    torch_dir = list(spec.submodule_search_locations)[0] if spec else None
    python_inc = sysconfig.get_paths()["include"]
    for what, path in (("torch", torch_dir), ("Python.h", os.path.join(python_inc, "Python.h")),
                       ("torch's C++ headers", torch_dir and os.path.join(torch_dir, "include", "torch", "csrc", "autograd", "python_variable.h"))):
        if not path or not os.path.exists(path):
            print(f"no native marshalling ({what} not found): calls from Python go through ctypes")
            return
    inc = [python_inc, os.path.join(torch_dir, "include"), os.path.join(torch_dir, "include", "torch", "csrc", "api", "include")]
    # the accessors of torch's tensor class are inlined: the binding uses the module with this torch only
    version = runpy.run_path(os.path.join(torch_dir, "version.py"))["__version__"]
    subprocess.check_call([HIPCC, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f'-DIG_BUILT_FOR="{version}"', *[f"-I{d}" for d in inc],
                           "-x", "c++", os.path.join(CSRC, "ig_call.cpp"), "-o", CALL, "-L" + os.path.join(torch_dir, "lib"),
                           "-ltorch_python", "-ltorch_cpu", "-lc10", "-L" + HERE, "-linfinigen_hip", "-Wl,-rpath,$ORIGIN"])


HOST_SANITIZED = ["ig_api.hip", "ig_host.cpp"]      # the files whose host code checks and computes


def sanitizer_runtime() -> str:
    """Path of the shared AddressSanitizer runtime of hipcc's clang (to be preloaded by a process
    that loads the host-sanitized library)."""
    clang = subprocess.check_output([HIPCC, "--hip-path=/opt/rocm", "-print-file-name=libclang_rt.asan-x86_64.so"],
                                    text=True).strip()
    if os.path.isabs(clang) and os.path.exists(clang):
        return clang
    import glob
    hits = sorted(glob.glob("/opt/rocm/lib/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so"))
    if not hits:
        raise FileNotFoundError("libclang_rt.asan-x86_64.so not found under /opt/rocm")
    return hits[-1]


def build_host_sanitized(out_dir: str) -> str:
    """Second copy of the library whose HOST code (argument checks, offline skewing, partial index,
    CPU-side speculation) is instrumented with AddressSanitizer and UndefinedBehaviorSanitizer;
    device code and the kernel launch files are the ordinary objects of build().  For the CPU test
    suite only."""
    os.makedirs(out_dir, exist_ok=True)
    san = ["-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=undefined"]
    objs = []
    for src in SOURCES:
        plain = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
        if src not in HOST_SANITIZED:
            if not os.path.exists(plain):
                _compile(src)
            objs.append(plain)
            continue
        obj = os.path.join(out_dir, os.path.splitext(src)[0] + ".o")
        path = os.path.join(CSRC, src)
        if src.endswith(".hip"):
            host = [f for flag in san for f in ("-Xarch_host", flag)]
            cmd = [HIPCC, "-O1", "-g", *COMMON[1:], *DEVICE_FLAGS, *host, "-c", path, "-o", obj]
        else:
            cmd = [HIPCC, "-O1", "-g", *COMMON[1:], *san, "-x", "c++", "-c", path, "-o", obj]
        subprocess.check_call(cmd)
        objs.append(obj)
    lib = os.path.join(out_dir, "libinfinigen_hip.so")
    subprocess.check_call([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-shared-libsan", *san, "-o", lib, *objs])
    return lib


if __name__ == "__main__":
    build(verbose=True)
