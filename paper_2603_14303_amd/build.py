"""Builds libsemanticache.so (HIP, gfx950) and the module _native (the argument marshalling of binding.py, C++) next to this file.

Usage: python -m paper_2603_14303_amd.build [--force]
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from importlib import metadata

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsemanticache.so")
NATIVE = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))      # (another Python looks for another name)
NATIVE_FOR = os.path.join(OBJ, "native_torch_version")                               # the torch that it was built against
SOURCES = ["sc_api.hip", "sc_segment.hip", "sc_gsc_merge.hip", "sc_gsc_fast.hip", "sc_gsc_global.hip", "sc_decode.hip", "sc_multi.hip", "sc_budget.hip", "sc_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed-fp32 instruction forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _deps():
    out = [os.path.join(CSRC, f) for f in os.listdir(CSRC)]
    out.append(os.path.join(os.path.dirname(HERE), "include", "semanticache.h"))
    return out


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, msgs))
    if msgs.strip():
        print(msgs, file=sys.stderr)
    return obj


def _torch_version():
    """The torch that is installed, or None."""
    try:
        return metadata.version("torch")
    except metadata.PackageNotFoundError:
        return None


def _newer_than_sources(out: str) -> bool:
    return os.path.exists(out) and all(os.path.getmtime(out) >= os.path.getmtime(d) for d in _deps())


def _native_is_current() -> bool:
    if _torch_version() is None:      # no torch, no wrappers
        return True
    if not (_newer_than_sources(NATIVE) and os.path.exists(NATIVE_FOR)):
        return False
    with open(NATIVE_FOR) as f:
        return f.read() == _torch_version()


def _build_native() -> None:
    """_native against the torch that is installed.  Without torch there are no wrappers to speed up; without a C++ compiler or the headers
    the wrappers marshal their calls in Python."""
    for old in (NATIVE, NATIVE_FOR):      # what is there was built from other sources, or against another torch
        if os.path.exists(old):
            os.remove(old)
    try:
        import torch
        from torch.utils.cpp_extension import include_paths
    except ImportError:
        return
    cxx, include = shutil.which("g++"), [*include_paths(), sysconfig.get_paths()["include"]]
    missing = [h for h in ("torch/csrc/autograd/python_variable.h", "ATen/core/Tensor.h", "Python.h") if not any(os.path.exists(os.path.join(i, h)) for i in include)]
    if cxx is None or missing:
        print("_native is not built: no %s" % (", ".join(missing) if cxx else "g++"), file=sys.stderr)
        return
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           '-DSC_TORCH_VERSION="%s"' % torch.__version__, *["-I" + i for i in include], os.path.join(CSRC, "sc_binding.cpp"), "-o", tmp,
           "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-L" + HERE, "-l:libsemanticache.so", "-Wl,-rpath,$ORIGIN"]
    subprocess.check_call(cmd)
    os.replace(tmp, NATIVE)
    with open(NATIVE_FOR, "w") as f:
        f.write(_torch_version() or "")


def build(force: bool = True) -> str:
    """Compile every HIP source for gfx950, link the shared library and build what binds it to Python.  Returns the library's path."""
    if not force and _newer_than_sources(LIB):
        if not _native_is_current():
            _build_native()
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    _build_native()
    return LIB


if __name__ == "__main__":
    print(build(force=True))
