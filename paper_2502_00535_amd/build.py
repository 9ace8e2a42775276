"""Compile the HIP library in-tree for gfx950 (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import warnings

_HERE = os.path.dirname(os.path.abspath(__file__))
SOURCES = [os.path.join(_HERE, "csrc", "nms_kernels.hip")]
HEADERS = [os.path.join(_HERE, "csrc", "nms_pair.h"), os.path.join(_HERE, "csrc", "nms_host_logic.h"), os.path.join(_HERE, "csrc", "nms_place.h"),
           os.path.join(os.path.dirname(_HERE), "include", "nms.h"),
           *sorted(os.path.join(_HERE, "csrc", "kernels", f)
                   for f in os.listdir(os.path.join(_HERE, "csrc", "kernels")) if f.endswith(".h"))]
LIBRARY = os.path.join(_HERE, "libnms_mi355x.so")
MARSHAL_SOURCE = os.path.join(_HERE, "csrc", "marshal.c")
MARSHAL = os.path.join(_HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))

# -ffp-contract=off: the pair test must round every operation on its own (the one
#   fused multiply-add it uses is written explicitly).
# -fno-honor-nans (device only): inputs are NaN-free by contract; without it every
#   min/max operand fetched from memory is first re-quieted with an extra VALU
#   instruction.  Host code keeps full NaN semantics for argument checking.
# -packed-fp32-ops off: no packed float32 VALU instructions are generated.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off",
    "-Xarch_device", "-fno-honor-nans",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def is_stale() -> bool:
    if not os.path.exists(LIBRARY):
        return True
    built = os.path.getmtime(LIBRARY)
    if any(os.path.getmtime(p) > built for p in SOURCES + HEADERS):
        return True
    return os.path.exists(MARSHAL) and os.path.getmtime(MARSHAL_SOURCE) > os.path.getmtime(MARSHAL)


def build_marshal() -> str:
    """The binding's native marshalling (CPython's C API, no device code); returns the path of the module."""
    tmp = MARSHAL + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"], MARSHAL_SOURCE, "-o", tmp]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("the C compiler failed:\n" + " ".join(cmd) + "\n" + proc.stdout + proc.stderr)
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build_marshal_if_possible() -> str | None:
    """The same where there is a C compiler and this Python's headers; without them the binding marshals every call in Python."""
    try:
        return build_marshal()
    except (OSError, RuntimeError) as e:
        if os.path.exists(MARSHAL):  # of an earlier state of its source
            os.remove(MARSHAL)
        warnings.warn(f"native marshalling not built, calls on small frames take 2 us longer: {e}")
        return None


def build_library(verbose: bool = False) -> str:
    """Always compiles (the binding's marshalling module as well, where that can be done); returns the path of the shared object."""
    build_marshal_if_possible()
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIBRARY + f".tmp{os.getpid()}"
    cmd = [hipcc, *HIPCC_FLAGS, *SOURCES, "-o", tmp]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + proc.stdout + proc.stderr)
    if verbose:
        # the host pass does not know the device-only target feature; that warning is expected
        print("\n".join(l for l in proc.stderr.splitlines() if "not a recognized feature" not in l))
    os.replace(tmp, LIBRARY)
    return LIBRARY


if __name__ == "__main__":
    print(build_library(verbose=True))
