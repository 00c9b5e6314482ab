"""Build the HIP library in-tree: csrc/*.hip -> libbtc_hip.so (gfx950 only), and the call path of the Python
binding: csrc/btc_python.c -> _native.so."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG), "include")
LIB = os.path.join(PKG, "libbtc_hip.so")
OBJ_DIR = os.path.join(PKG, "_build")
NATIVE = os.path.join(PKG, "_native.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources() -> list[str]:
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd: list[str]) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + err)
    return err


def build(verbose: bool = False, incremental: bool = False, jobs: int = 8) -> str:
    """Compile every source (one object per file, `jobs` at a time) and link.  Every call compiles everything
    unless `incremental` is set, which skips objects newer than their source and every header."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    headers = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    newest_header = max(os.path.getmtime(h) for h in headers)
    todo, objs = [], []
    for src in sources():
        obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        if incremental and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header):
            continue
        todo.append([hipcc, *HIPCC_FLAGS, *os.environ.get("BTC_EXTRA_HIPCC_FLAGS", "").split(), "-I", INCLUDE, "-I", CSRC, "-c", "-o", obj, src])
    with concurrent.futures.ThreadPoolExecutor(max_workers=max(1, jobs)) as pool:
        for cmd, err in zip(todo, pool.map(_run, todo)):
            if verbose:
                print(" ".join(cmd))
                if err.strip():
                    print(err)
    err = _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    if verbose and err.strip():
        print(err)
    native_src = os.path.join(CSRC, "btc_python.c")
    if not (incremental and os.path.exists(NATIVE) and os.path.getmtime(NATIVE) > os.path.getmtime(native_src)):
        err = _run([os.environ.get("CC", "gcc"), "-O2", "-Wall", "-Wextra", "-shared", "-fPIC", "-fvisibility=hidden",
                    "-I", sysconfig.get_paths()["include"], "-o", NATIVE, native_src])
        if verbose and err.strip():
            print(err)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose=True, incremental="--incremental" in sys.argv))
