"""Build libsv.so (HIP, gfx950) in-tree with hipcc.

Every source under csrc/ is compiled for gfx950 only and linked into
paper_1805_00988_amd/libsv.so, which the Python binding loads.
"""

from __future__ import annotations

import json
import os
import re
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libsv.so")
# uses the struct layouts of the interpreter that builds it: tagged with its ABI
PY_OUT = os.path.join(HERE, "libsvpy" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
OBJ = os.path.join(HERE, "_build")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
    "-Wno-unused-result",
    # packed-FP32 instructions are kept out of all generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics",
    # uniform (scalar) branches are left unstructured: the sweep kernels'
    # per-gate dispatch then merges its paths without copying the register
    # group held across it
    "-mllvm", "-structurizecfg-skip-uniform-regions=true",
    # per-kernel register / scratch / occupancy report (parsed into _build/)
    "-Rpass-analysis=kernel-resource-usage",
]
RESOURCES = os.path.join(OBJ, "kernel_resources.json")


def parse_resources(text: str) -> dict:
    """Kernel resource remarks -> {kernel: {field: int}}."""
    out, cur = {}, None
    for line in text.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark: \s*([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", line)
        if m and cur is not None:
            cur[m.group(1).strip()] = int(m.group(2))
    return out


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    cc = hipcc()
    srcs = sources()

    def compile_one(src):
        obj = os.path.join(OBJ, os.path.basename(src) + ".o")
        cmd = [cc, *HIPCC_FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        return obj, parse_resources(r.stderr)

    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        results = list(ex.map(compile_one, srcs))
    objs = [o for o, _ in results]
    resources = {}
    for _, res in results:
        resources.update(res)
    with open(RESOURCES, "w") as f:
        json.dump(resources, f, indent=1, sort_keys=True)
    spills = {k: v for k, v in resources.items() if v.get("ScratchSize", 0) > 0}
    if spills:
        print(f"warning: kernels using scratch memory: {sorted(spills)}", file=sys.stderr)
    tmp = OUT + ".tmp"
    cmd = [cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    build_py()
    return OUT


def build_py() -> str:
    """The binding's C helper (host code of the running interpreter's ABI).
    Without the interpreter's headers or a C++ compiler there is none ('' is
    returned, and an earlier one is removed): the binding then converts gate
    lists in Python."""
    include = sysconfig.get_paths()["include"]
    cxx = shutil.which(os.environ.get("CXX") or "g++")
    if cxx is None or not os.path.exists(os.path.join(include, "Python.h")):
        print(f"note: {os.path.basename(PY_OUT)} is not built (no C++ compiler or no Python.h)", file=sys.stderr)
        if os.path.exists(PY_OUT):
            os.remove(PY_OUT)
        return ""
    tmp = PY_OUT + ".tmp"
    cmd = [cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I" + include, os.path.join(CSRC, "py_ops.cpp"),
           "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building {PY_OUT} failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, PY_OUT)
    return PY_OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
