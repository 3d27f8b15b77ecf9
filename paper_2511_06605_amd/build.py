"""Build the HIP library in-tree for gfx950 (explicit hipcc, no JIT cache)."""

from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdmalatte.so")
# (with the tag of the Python it is built for: no other one loads it)
MARSHAL = os.path.join(HERE, "_marshal" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["dl_api.hip", "dl_exec.hip", "dl_prelaunch.hip", "dl_dispatch.hip", "dl_static.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # packed-fp32 instructions stay off for every device function in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    # the host pass does not know the packed-fp32 feature and says so once per function
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if err:
        print(err, file=sys.stderr, flush=True)
    if r.returncode:
        raise subprocess.CalledProcessError(r.returncode, cmd)


def _build_marshal(verbose) -> None:
    """The extension module that marshals Python arguments for the library, if this Python's headers are here.  Without
    them the package makes the same calls with ctypes objects (marshal_ctypes.py); programs in C need neither."""
    for old in (MARSHAL, os.path.join(HERE, "_marshal.so")):
        if os.path.exists(old):
            os.remove(old)
    include = sysconfig.get_paths()["include"]
    cc = os.environ.get("CC") or next(filter(None, map(shutil.which, ("gcc", "cc", "/opt/rocm/llvm/bin/clang"))), None)
    if not cc or not os.path.exists(os.path.join(include, "Python.h")):
        print(f"no {'Python headers in ' + include if cc else 'C compiler'}: without the marshalling module, Python calls take longer",
              file=sys.stderr, flush=True)
        return
    _run([*cc.split(), "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-Wextra", "-Wno-unused-parameter",
          "-Wno-missing-field-initializers", "-I" + include, os.path.join(CSRC, "dl_marshal.c"), "-o", MARSHAL], verbose)


def build(verbose: bool = False) -> str:
    """The library, then the extension module for Python."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc, *HIPCC_FLAGS, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB], verbose)
    _build_marshal(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
