"""Build the HIP library liblbrr.so in-tree for gfx950 (hipcc, no GPU needed).

Usage: python -m paper_1505_06900_amd.build [-j JOBS] [--verbose] [--sanitized DIR]

--sanitized DIR also writes DIR/liblbrr_asan.so: the same library with its host
code built with AddressSanitizer and UndefinedBehaviorSanitizer (the GPU code is
the normal build's, taken from its objects), for host-side tests on the CPU with
the sanitizer runtime preloaded (sanitizer_runtime()).
"""
from __future__ import annotations

import argparse
import concurrent.futures as cf
import json
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "liblbrr.so")
# per-kernel register, scratch, LDS and occupancy figures reported by the compiler
RESOURCES = os.path.join(PKG, "liblbrr_resources.json")

SOURCES = ["api.hip", "diag.hip", "probe.hip", "closure.hip", "kernels_d2q9.hip", "kernels_d3q19.hip", "kernels_d3q27.hip",
           "kernels_pair_d2q9.hip", "kernels_pair_d3q19.hip", "kernels_pair_d3q27.hip"]

ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-ffp-contract=fast",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    # per-kernel resource usage as compiler remarks (analysis only; collected into RESOURCES)
    "-Rpass-analysis=kernel-resource-usage",
]

# per-source additions: the closure kernels take matrix-core results in ordinary
# VGPRs, so the activations read them without a copy from the accumulation registers
SOURCE_FLAGS = {"closure.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def parse_resource_remarks(text):
    """{kernel name: {field: value}} from the compiler's kernel-resource-usage remarks."""
    out, cur = {}, None
    for line in text.splitlines():
        if "remark:" not in line or "kernel-resource-usage" not in line:
            continue
        body = line.split("remark:", 1)[1].rsplit("[-Rpass-analysis", 1)[0].strip()
        key, _, val = body.partition(":")
        key, val = key.strip(), val.strip()
        if key == "Function Name":
            cur = out.setdefault(val, {})
        elif cur is not None and val:
            cur[key] = int(val) if val.lstrip("-").isdigit() else val
    return out


def demangle(names):
    exe = shutil.which("c++filt") or shutil.which("llvm-cxxfilt")
    if not exe or not names:
        return {n: n for n in names}
    r = subprocess.run([exe], input="\n".join(names), capture_output=True, text=True)
    out = r.stdout.splitlines() if r.returncode == 0 else []
    return dict(zip(names, out)) if len(out) == len(names) else {n: n for n in names}


def hipcc():
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found (ROCm toolchain required to build liblbrr.so)")
    return exe


def _compile(src, verbose):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc(), *FLAGS, *SOURCE_FLAGS.get(src, []), "-I", os.path.join(ROOT, "include"), "-c",
           os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj, r.stderr


def build(jobs=None, verbose=False):
    """Compile every source and link liblbrr.so.  Always recompiles."""
    os.makedirs(BUILD, exist_ok=True)
    jobs = jobs or min(len(SOURCES), max(1, (os.cpu_count() or 2)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    objs = [o for o, _ in results]
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    res = {}
    for _, err in results:
        res.update(parse_resource_remarks(err))
    names = demangle(sorted(res))
    with open(RESOURCES, "w") as fh:
        json.dump({names[k]: v for k, v in sorted(res.items())}, fh, indent=1)
    return LIB


def _llvm_tool(name):
    exe = os.path.join(os.path.dirname(os.path.realpath(hipcc())), "..", "llvm", "bin", name)
    exe = exe if os.path.exists(exe) else os.path.join("/opt/rocm/llvm/bin", name)
    if not os.path.exists(exe):
        raise RuntimeError(f"{name} not found")
    return exe


def sanitizer_runtime():
    """Path of the AddressSanitizer runtime of the ROCm compiler (it carries the UBSan handlers), or None."""
    import glob

    hits = sorted(glob.glob("/opt/rocm/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so"))
    return hits[-1] if hits else None


SANITIZE = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
            "-Xarch_host", "-fno-omit-frame-pointer"]


def build_sanitized(out_dir, jobs=None):
    """Host code under ASan + UBSan, GPU code from the normal build's objects (build() first).

    Each source's host part is compiled alone (--offload-host-only) with the GPU
    binary that build() embedded in its object passed back in, so the GPU code is
    not compiled again."""
    os.makedirs(out_dir, exist_ok=True)
    objcopy = _llvm_tool("llvm-objcopy")

    def one(src):
        stem = os.path.splitext(src)[0]
        normal = os.path.join(BUILD, stem + ".o")
        if not os.path.exists(normal):
            raise RuntimeError(f"{normal} is missing: run build() first")
        fatbin = os.path.join(out_dir, stem + ".fatbin")
        subprocess.run([objcopy, "-O", "binary", "--only-section=.hip_fatbin", normal, fatbin], check=True)
        obj = os.path.join(out_dir, stem + ".o")
        cmd = [hipcc(), f"--offload-arch={ARCH}", "--offload-host-only", "-Xclang", "-fcuda-include-gpubinary",
               "-Xclang", fatbin, "-O1", "-g", "-std=c++17", "-fPIC", "-Wno-unused-command-line-argument", *SANITIZE,
               "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"sanitized host compile failed for {src}:\n{r.stderr}")
        return obj

    jobs = jobs or min(len(SOURCES), max(1, (os.cpu_count() or 2)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(one, SOURCES))
    lib = os.path.join(out_dir, "liblbrr_asan.so")
    cmd = [hipcc(), f"--offload-arch={ARCH}", "--offload-host-only", "-shared", "-fPIC", *objs, *SANITIZE, "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"sanitized link failed:\n{r.stderr}")
    return lib


def main(argv=None):
    ap = argparse.ArgumentParser()
    ap.add_argument("-j", "--jobs", type=int, default=None)
    ap.add_argument("--verbose", action="store_true")
    ap.add_argument("--sanitized", metavar="DIR", default=None)
    a = ap.parse_args(argv)
    print(build(a.jobs, a.verbose))
    if a.sanitized:
        print(build_sanitized(a.sanitized, a.jobs))


if __name__ == "__main__":
    sys.exit(main())
