"""Build libhq.so (gfx950 kernels + host plan + C ABI) in-tree with hipcc.

    python -m paper_2606_23406_amd.build
"""
import hashlib
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhq.so")
SOURCES = [os.path.join(CSRC, f) for f in ("hq_encode.hip", "hq_decode.hip", "hq_fused.hip", "hq_gemm.hip",
                                          "hq_host.cpp")]
DEPS = SOURCES + [os.path.join(CSRC, "hq_internal.h"), os.path.join(CSRC, "hq_device.h"),
                  os.path.join(CSRC, "hq_lds.h"), os.path.join(CSRC, "calib_table.inc"),
                  os.path.join(os.path.dirname(HERE), "include", "hq.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # every fp32 rounding in the kernels is the one written; no fused contractions
    "-ffp-contract=off",
    # no packed fp32 vector instructions (v_pk_*_f32) are generated
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def source_sha256() -> str:
    """Hash of the sources a library is built from (a measurement's stamp)."""
    h = hashlib.sha256()
    for d in sorted(DEPS):
        h.update(open(d, "rb").read())
    return h.hexdigest()


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(d) > t for d in DEPS)


def build(verbose: bool = False) -> str:
    # one object per source, compiled side by side, then linked
    tmp = LIB + ".tmp"
    objs = [LIB + "." + os.path.basename(s) + ".o" for s in SOURCES]
    cmds = [[HIPCC] + FLAGS + ["-c", "-o", o, s] for o, s in zip(objs, SOURCES)]
    link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed building libhq.so")

    try:
        with ThreadPoolExecutor(len(cmds)) as pool:
            list(pool.map(run, cmds))
        run(link)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
