"""Build the gfx950 HIP library ``libcatalan.so`` in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcatalan.so")
SOURCES = ["catalan.hip", "fntt.hip"]   # compiled side by side, then linked
DEPS = ["catalan.hip", "fntt.hip", "fntt.hpp", "common.hpp", "ntt.inc.hip", "small.inc.hip", "fused.inc.hip", "sieve.inc.hip", "ratio.inc.hip",
        "decimal.inc.hip", "host.inc.hip", "decimal_host.inc.hip", "rates.inc.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # no packed FP32 instructions anywhere in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def needs_build() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, d) for d in DEPS]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "catalan.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def _run(cmds, verbose: bool) -> None:
    """The commands side by side; raises with their output if one fails."""
    procs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append(subprocess.Popen(cmd, cwd=CSRC, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    outs = [p.communicate()[0] for p in procs]
    if any(p.returncode for p in procs):
        sys.stderr.write("\n".join(l for o in outs for l in o.splitlines() if "packed-fp32-ops" not in l) + "\n")
        raise RuntimeError("hipcc failed building libcatalan.so")


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not needs_build():
        return LIB
    tmp = LIB + ".tmp%d" % os.getpid()
    objs = [tmp + "." + src.split(".")[0] + ".o" for src in SOURCES]
    cmds = [[HIPCC] + FLAGS + ["-c", "-o", o, os.path.join(CSRC, src)] for o, src in zip(objs, SOURCES)]
    link = [HIPCC] + FLAGS + ["-shared", "-o", tmp] + objs
    try:
        _run(cmds, verbose)
        _run([link], verbose)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
