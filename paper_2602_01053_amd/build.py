"""Compile the HIP library for gfx950 and the CPython module that calls it, in-tree."""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "liblra_attn.so")
PYCALL_SOURCE = "lra_pycall.cpp"   # CPython module over the C ABI, on its own: it links neither the library nor torch
# (named for the interpreter that it is compiled for: it uses more than the stable ABI, and no other one may load it)
PYCALL_PATH = os.path.join(PKG_DIR, "_lra_pycall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
# what the compiler reports per kernel (registers, scratch, LDS, occupancy), written by every build
RESOURCES_PATH = os.path.join(PKG_DIR, "kernel_resources.json")

SOURCES = ["lra_plan.cpp", "lra_api.hip", "lra_generic.hip", "lra_decode_mfma.hip", "lra_decode_batch.hip", "lra_decode_stream.hip", "lra_prefill_mfma.hip", "lra_prefill_rows.hip", "lra_append.hip", "lra_probe.hip"]

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    # packed fp32 instructions are kept out of every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # the LDS transfers set M0 inside their assembly statement and say so in the clobber list
    "-Wno-inline-asm",
]
# (device pass only) one remark block per kernel with its register, scratch and LDS use
RESOURCE_REMARKS = "-Rpass-analysis=kernel-resource-usage"


def source_fingerprint() -> str:
    """Hash (16 hex digits) of everything the library is compiled from: the sources, the headers
    beside them and the public headers.  Measurements kept next to the code (HBM traffic per launch
    from hardware counters) record it, so that a reader can tell whether they were taken on these
    kernels or on earlier ones."""
    import hashlib
    h = hashlib.sha256()
    inc = os.path.join(ROOT, "include")
    files = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith((".hip", ".h", ".cpp"))]
    files += [os.path.join(inc, f) for f in sorted(os.listdir(inc)) if f.endswith(".h")]
    for path in files:
        h.update(os.path.basename(path).encode())
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def _parse_resource_remarks(stderr: str) -> dict:
    """{mangled kernel name: {"VGPRs": .., "AGPRs": .., "ScratchSize [bytes/lane]": .., ...}} from the
    compiler's kernel-resource-usage remarks."""
    out, cur = {}, None
    for ln in stderr.splitlines():
        if "[-Rpass-analysis=kernel-resource-usage]" not in ln:
            continue
        m = re.search(r"remark:\s+Function Name: (\S+)", ln)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+([^:]+): (\S+) \[-Rpass", ln)
        if m and cur is not None:
            v = m.group(2)
            cur[m.group(1).strip()] = int(v) if v.isdigit() else v
    return out


def _run(cmd, verbose):
    """Runs one compiler command; returns the kernel resource table its remarks hold (empty for host code)."""
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    remarks, rest, skip = [], [], 0
    for ln in res.stderr.splitlines():
        if "[-Rpass-analysis=kernel-resource-usage]" in ln:
            remarks.append(ln)
            skip = 2 if "Function Name" in ln else 0  # (the first remark of a kernel is followed by its source line and a caret)
        elif skip > 0 and re.match(r"^\s+(\d+ \||\|)", ln):
            skip -= 1
        elif "packed-fp32-ops" not in ln:
            rest.append(ln)
    err = "\n".join(rest)
    if res.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed ({res.returncode}): {' '.join(cmd)}\n{err}")
    if verbose and err.strip():
        print(err)
    return _parse_resource_remarks("\n".join(remarks))


def build_library(verbose: bool = False) -> str:
    """Compile every source to an object file (in parallel, under _build/), link the shared library, and build the
    CPython module that calls it (build_pycall)."""
    from concurrent.futures import ThreadPoolExecutor
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj_dir = os.path.join(ROOT, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    jobs = []
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        if not os.path.exists(path):
            raise FileNotFoundError(path)
        obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
        if src.endswith(".cpp"):   # host-only C++ (launch planning): no device pass
            jobs.append(([hipcc, "-O2", "-std=c++17", "-fPIC", *inc, "-c", path, "-o", obj], obj))
        else:
            jobs.append(([hipcc, *HIPCC_FLAGS, RESOURCE_REMARKS, *inc, "-c", path, "-o", obj], obj))
    with ThreadPoolExecutor(max_workers=min(len(jobs), os.cpu_count() or 1)) as pool:
        tables = list(pool.map(lambda j: _run(j[0], verbose), jobs))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *[o for _, o in jobs], "-o", LIB_PATH], verbose)
    import json
    resources = {}
    for (cmd, _), table in zip(jobs, tables):
        for name, row in table.items():
            resources[name] = dict(row, source=os.path.basename(cmd[-3]))
    with open(RESOURCES_PATH, "w") as f:
        json.dump({"source_fingerprint": source_fingerprint(), "kernels": resources}, f, indent=0, sort_keys=True)
    build_pycall(hipcc, verbose)
    return LIB_PATH


def build_pycall(hipcc: str, verbose: bool = False) -> bool:
    """Compile the CPython module, with the host compiler or else with hipcc's.  Without the interpreter's headers there is
    none, nor one left from an earlier build: the binding then makes its calls by ctypes."""
    headers = sysconfig.get_paths()["include"]
    if os.path.exists(PYCALL_PATH):
        os.remove(PYCALL_PATH)
    if not os.path.exists(os.path.join(headers, "Python.h")):
        print(f"no Python.h under {headers}: calls go through ctypes", flush=True)
        return False
    cxx = os.environ.get("CXX") or shutil.which("g++") or hipcc
    _run([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-I", headers, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          os.path.join(CSRC, PYCALL_SOURCE), "-o", PYCALL_PATH], verbose)
    return True


if __name__ == "__main__":
    print(build_library(verbose=True))
