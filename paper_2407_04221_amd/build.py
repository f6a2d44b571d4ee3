"""Build libautoverse.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libautoverse.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["av_api.cpp", "av_search.cpp", "k_generic.hip", "k_wave.hip", "k_rows.hip", "k_observe.hip",
           "k_mutate.hip", "k_search.hip", "jit.cpp", "lane16_jit.cpp", "av_static.cpp",
           "k_group.hip"]
TEMPLATE = "lane16_kernel.hip"          # compiled at run time, per rule set, with hipRTC
# Device code is built without packed-FP32 instructions.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def embed_template() -> None:
    """Write the lane16 kernel template into a C++ string the library compiles in."""
    text = open(os.path.join(CSRC, TEMPLATE)).read()
    assert ")AVK\"" not in text
    philox = open(os.path.join(CSRC, "philox.h")).read()
    assert ")AVK\"" not in philox
    with open(os.path.join(CSRC, "_lane16_template.inc"), "w") as f:
        f.write("// generated by build.py from lane16_kernel.hip and philox.h; do not edit\n")
        f.write('static const char kLane16Template[] = R"AVK(' + text + ')AVK";\n')
        f.write('static const char kPhiloxSource[] = R"AVK(' + philox + ')AVK";\n')


def check_template(verbose: bool = False) -> None:
    """The template alone (no rules) must compile for gfx950."""
    obj = os.path.join(CSRC, "_lane16_check.o")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-c",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           os.path.join(CSRC, TEMPLATE), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True, cwd=CSRC)
    os.remove(obj)


def build(out: str = LIB, verbose: bool = False) -> str:
    embed_template()
    check_template(verbose)
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    cmd = [HIPCC, *FLAGS, "-x", "hip", *srcs, "-lhiprtc", "-o", out + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True, cwd=CSRC)
    os.replace(out + ".tmp", out)
    return out


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
