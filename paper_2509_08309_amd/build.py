"""Build libhetis_attn.so for gfx950 with hipcc and the binding's argument marshalling (_marshal.so, host
code), in-tree (next to this file)."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhetis_attn.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
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


def is_current() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(MARSHAL)):
        return False
    t = min(os.path.getmtime(LIB), os.path.getmtime(MARSHAL))
    return all(os.path.getmtime(s) <= t for s in sources())


def build(force: bool = True, extra_flags=()) -> str:
    if not force and is_current():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + \
          [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL],
                   check=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(extra_flags=sys.argv[1:]))
