"""Build the gfx950 HIP library (librkc.so) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRCS = [os.path.join(PKG, "csrc", f) for f in ("rkc_replay.hip", "rkc_lean.hip", "rkc_lean_few.hip",
                                              "rkc_big.hip", "rkc_tiny.hip")]
LIB = os.path.join(PKG, "librkc.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed FP32 instructions are kept off for all device code on this hardware
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # Leave regions whose branches are wave-uniform unstructured.  The per-pool event loops branch
    # only on wave-uniform values; structurizing those regions merged the outputs of two branches of
    # a refusal wrongly in some builds (a capacity refusal's b came out as the other branch's value),
    # which no build with this setting shows.
    "-mllvm", "-structurizecfg-skip-uniform-regions=true",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
    "-I", os.path.join(ROOT, "include"),
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


# checking build: every readfirstlane also verifies that the active lanes agree (slower; used to
# run the GPU parity suite once against the uniformity assumptions of both kernels)
CHECK_LIB = os.path.join(PKG, "librkc_check.so")


# Kernels that address their dynamic LDS from 0 (lat() in rkc_lean.hip and rkc_big.hip), where it starts only
# while they have no static LDS: a __shared__ variable in one of them would share its bytes with the pool's state.
LDS_FROM_ZERO = re.compile(r"\d(rkc_lean|rkc_big)[IE]")
RESOURCES = ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics"]


def static_lds(remarks: str) -> dict[str, int]:
    """Bytes of static LDS per kernel (mangled name), from the compiler's resource remarks."""
    name, out = None, {}
    for line in remarks.splitlines():
        m = re.search(r"remark:\s+(Function Name|LDS Size \[bytes/block\]): (\S+)", line)
        if m and m[1] == "Function Name":
            name = m[2]
        elif m and name:
            out[name] = int(m[2])
    return out


def compile_source(src: str, obj: str, flags: list[str]) -> None:
    """Compile one source; refuse an object whose kernels' LDS does not start where they take it to."""
    r = subprocess.run([*flags, *RESOURCES, "-c", src, "-o", obj], stderr=subprocess.PIPE, text=True)
    sys.stderr.write("".join(x for x in r.stderr.splitlines(keepends=True) if RESOURCES[0] not in x))
    if r.returncode:
        raise subprocess.CalledProcessError(r.returncode, r.args)
    lds = static_lds(r.stderr)
    bad = [k for k, n in lds.items() if n and LDS_FROM_ZERO.search(k)]
    if bad or not lds:
        os.unlink(obj)
        raise RuntimeError(f"{src}: static LDS in kernels that address dynamic LDS from 0: {bad}" if bad else
                           f"{src}: the compiler reported no kernel's resources")


def build(verbose: bool = False, check_uniform: bool = False) -> str:
    out = CHECK_LIB if check_uniform else LIB
    tmp = out + ".tmp%d" % os.getpid()
    flags = [hipcc(), *HIPCC_FLAGS, *(["-DRKC_CHECK_UNIFORM"] if check_uniform else [])]
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, os.path.basename(f) + ".o") for f in SRCS]
        link = [hipcc(), "-shared", f"--offload-arch={ARCH}", *objs, "-o", tmp]
        if verbose:
            print("\n".join(" ".join(c) for c in [*([*flags, "-c", f, "-o", o] for f, o in zip(SRCS, objs)), link]), flush=True)
        # the sources are independent: one compiler each, side by side
        with ThreadPoolExecutor(min(len(objs), os.cpu_count() or 1)) as pool:
            list(pool.map(lambda f, o: compile_source(f, o, flags), SRCS, objs))
        subprocess.check_call(link)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose=True, check_uniform="--check-uniform" in sys.argv))
