"""Build libsllg.so (HIP kernels + C++ runtime + C ABI) for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libsllg.so")
SOURCES = ["kernels.hip", "fused.hip", "brick.hip", "longrange.hip", "noalloc.hip", "prepare.cpp", "api.cpp", "server.cpp", "builders.cpp"]

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    "-Wall", "-Wno-unused-function",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-pthread",
]


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source into paper_1310_6143_amd/libsllg.so (always
    recompiles when force is true)."""
    if not force and os.path.exists(LIB_PATH):
        return LIB_PATH
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    tmp = LIB_PATH + ".tmp"
    with tempfile.TemporaryDirectory() as objs:   # one compiler per source, then the link
        jobs = []
        for s in srcs:
            o = os.path.join(objs, os.path.basename(s) + ".o")
            jobs.append((o, subprocess.Popen([hipcc] + HIPCC_FLAGS + ["-c", s, "-o", o], text=True,
                                             stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        out = [p.communicate()[0] for _, p in jobs]
        if any(p.returncode for _, p in jobs):
            raise RuntimeError("hipcc failed:\n" + "".join(out))
        res = subprocess.run([hipcc] + HIPCC_FLAGS + ["-shared"] + [o for o, _ in jobs] + ["-o", tmp],
                             capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print("".join(out))
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
