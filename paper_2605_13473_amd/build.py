"""Build libosdn.so (the HIP library) in-tree for gfx950 with hipcc, and the extension module _native (binding.step's way to it)
with g++.  The library needs hipcc alone: without g++ or the headers of Python and the tensor library it is built, and
the module, which only saves time, is not (binding.step then goes through Python, and says so)."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libosdn.so")
NATIVE = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))     # (the name says for which Python)
NATIVE_SOURCE = os.path.join(CSRC, "osdn_native.cpp")
SOURCES = ["osdn_api.hip", "osdn_precond.hip", "osdn_precond_bwd.hip", "osdn_precond_gen.hip", "osdn_step.hip", "osdn_tables.hip",
           "osdn_chunk_fwd.hip", "osdn_chunk_bwd.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False, only=None) -> str:
    """Compile every HIP source of the library (side by side, one hipcc per file) and link
    them into one shared object.  `only`: recompile just these sources and reuse the other
    objects of an earlier build (for quick iteration; the default compiles everything)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)

    # an object is reused only if it is newer than every header (the kernels pass their arguments
    # in structs declared there: an object built against an older layout must never be linked)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    headers.append(os.path.join(os.path.dirname(HERE), "include", "osdn.h"))
    newest_header = max(os.path.getmtime(h) for h in headers if os.path.exists(h))

    def compile_one(src):
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        if (only is not None and src not in only and os.path.exists(obj)
                and os.path.getmtime(obj) > max(newest_header, os.path.getmtime(os.path.join(CSRC, src)))):
            return obj
        cmd = [hipcc, *FLAGS, "-c", "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd))
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0 or verbose:
            print(r.stdout)
        if r.returncode != 0:
            raise subprocess.CalledProcessError(r.returncode, cmd)
        return obj

    with ThreadPoolExecutor(max_workers=8) as pool:
        native = None if only is not None and native_is_current() else pool.submit(build_native)
        objs = list(pool.map(compile_one, SOURCES))
        if native is not None:
            native.result()
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


def native_is_current() -> bool:
    """The rule of the objects: the module fills a struct of osdn.h."""
    sources = (NATIVE_SOURCE, os.path.join(os.path.dirname(HERE), "include", "osdn.h"))
    return os.path.exists(NATIVE) and os.path.getmtime(NATIVE) > max(os.path.getmtime(f) for f in sources)


def build_native():
    """The extension module: host code alone, against the tensor library's headers.  Returns its path, or None, with a word of why, where it
    cannot be built; what stood there before is gone then."""
    for old in glob.glob(os.path.join(HERE, "_native*.so")):
        os.remove(old)
    try:
        import torch
        root = os.path.dirname(torch.__file__)
        lib = os.path.join(root, "lib")
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
               f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DOSDN_TORCH_VERSION="{torch.__version__}"',
               "-I" + sysconfig.get_paths()["include"],
               "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
               "-o", NATIVE, NATIVE_SOURCE, "-L" + lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        why = r.stdout if r.returncode != 0 else None
    except (ImportError, OSError) as e:
        why = str(e)
    if why is None:
        return NATIVE
    print(why)
    warnings.warn("the extension module was not built: binding.step goes through Python, at twice the time of a small call")
    return None


if __name__ == "__main__":
    import sys
    print(build(verbose=True, only=sys.argv[1:] or None))
