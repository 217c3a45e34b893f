"""Build libhetis_attn.so for gfx950 with hipcc and the binding's argument marshalling (host code, an extension
of the interpreter that runs this), in-tree (next to this file)."""
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhetis_attn.so")
# (the name carries the interpreter's version: another one does not pick up what it cannot load)
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["hetis_attn.hip", "hetis_kv.hip", "hetis_profiler.hip", "hetis_dispatch.hip"]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    out = []
    for root, _, files in os.walk(CSRC):
        out += [os.path.join(root, f) for f in files if f.endswith((".hip", ".hpp", ".h", ".cpp"))]
    inc = os.path.join(os.path.dirname(HERE), "include")
    out += [os.path.join(inc, f) for f in ("hetis_attn.h", "hetis_kv.h", "hetis_profiler.h", "hetis_dispatch.h")]
    return out


def marshal_compiler():
    """The C++ compiler of the marshalling extension; None where it or Python's headers are missing, and the
    binding then converts arguments through ctypes."""
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return None
    return os.environ.get("CXX") or shutil.which("g++")


def is_current() -> bool:
    built = [LIB, MARSHAL] if marshal_compiler() else [LIB]
    if not all(os.path.exists(b) for b in built):
        return False
    t = min(os.path.getmtime(b) for b in built)
    return all(os.path.getmtime(s) <= t for s in sources())


def build(force: bool = True, extra_flags=()) -> str:
    if not force and is_current():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + \
          [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    if marshal_compiler():
        subprocess.run([marshal_compiler(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                        "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL],
                       check=True)
    else:
        print("no C++ compiler or no Python headers: the binding converts arguments through ctypes", file=sys.stderr)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(extra_flags=sys.argv[1:]))
