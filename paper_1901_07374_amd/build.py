"""Build libtlsph.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libtlsph.so")
CSRC = os.path.join(HERE, "csrc")
# sources, each with flags of its own
SOURCES = {
    "tlsph_kernels.hip": [],
    # constants (the 64-bit literals of exp and log) are formed where they are
    # used: hoisted out of loops they take registers these kernels do not have
    "tlsph_passes_full.hip": ["-mllvm", "-disable-machine-licm"],
    "tlsph_host.hip": [],
}
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # no implicit multiply-add fusion: the hot loops spell out their fma()
    # calls, so every kernel variant rounds the same arithmetic the same way
    "-ffp-contract=off",
    # packed FP32 instructions stay off in all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        cmds, objs = [], []
        for name, extra in SOURCES.items():
            objs.append(os.path.join(tmp, name + ".o"))
            cmds.append([HIPCC, *FLAGS, *extra, "-c", "-o", objs[-1], os.path.join(CSRC, name)])
        jobs = [subprocess.Popen(c) for c in cmds]
        for cmd, code in zip(cmds, [job.wait() for job in jobs]):
            if verbose:
                print(" ".join(cmd), flush=True)
            if code:
                raise subprocess.CalledProcessError(code, cmd)
        link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB + ".tmp", *objs]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.check_call(link)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)


def source_hash() -> str:
    """Short digest of the device sources: counter summaries taken on other
    sources are recognised as stale."""
    import hashlib
    h = hashlib.sha1()
    for f in ("tlsph_kernels.hip", "tlsph_passes_full.hip", "tlsph_passes.h", "tlsph_math.h",
              "tlsph_internal.h"):
        with open(os.path.join(HERE, "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]
