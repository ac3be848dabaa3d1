"""Builds libmh3d.so (the C ABI of include/mh3d.h) in-tree with hipcc for gfx950."""
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libmh3d.so")
SOURCES = [os.path.join(PKG, "csrc", f) for f in ("mh3d.hip", "sep.hip", "fast.hip", "user.hip", "user_class1.hip",
                                                       "user_class2.hip", "user_class4.hip", "user_class3689.hip")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions are disabled for every HIP translation unit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
]


def build(verbose=True, extra=()):
    """Compile the library; raises CalledProcessError on failure."""
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        return subprocess.Popen(cmd), cmd

    def wait(started):
        for p, cmd in [(p, cmd) for p, cmd in started if p.wait() != 0]:
            raise subprocess.CalledProcessError(p.returncode, cmd)

    objs = [src[:-len(".hip")] + ".o" for src in SOURCES]     # the units compile side by side
    wait([run([HIPCC] + FLAGS + list(extra) + ["-c", src, "-o", obj]) for src, obj in zip(SOURCES, objs)])
    tmp = LIB + ".tmp"
    wait([run([HIPCC, "--offload-arch=gfx950", "-shared"] + objs + ["-o", tmp])])
    os.replace(tmp, LIB)
    for obj in objs:
        os.remove(obj)
    return LIB


if __name__ == "__main__":
    build(extra=sys.argv[1:])
