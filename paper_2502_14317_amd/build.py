"""Builds libparallelcomp.so (hand-written HIP for gfx950) in-tree with hipcc."""
import importlib.util
import os
import subprocess
import sys

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG_DIR), "include")
LIB_PATH = os.path.join(PKG_DIR, "libparallelcomp.so")
SOURCES = ["pc_api.hip", "prep.hip", "gather.hip", "select.hip", "decode_attn.hip", "prefill_attn.hip",
           "scores.hip", "ceiling.hip", "self_info.hip", "decode_attn_fp8.hip"]
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wno-unused-command-line-argument",
               # keep MFMA results in architectural VGPRs where the vector ALU consumes them
               # (softmax of S^T): avoids hundreds of accumulator<->VGPR copies per tile
               "-mllvm", "-amdgpu-mfma-vgpr-form=1"]


# Its assembly text is checked before the library is linked; the compiler leaves what it assembled beside the object
CHECKED = "prefill_attn.hip"


def check_spacing(obj_dir: str) -> None:
    spec = importlib.util.spec_from_file_location("spacing", os.path.join(PKG_DIR, "spacing.py"))
    spacing = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(spacing)
    with open(os.path.join(obj_dir, CHECKED.replace(".hip", "-hip-amdgcn-amd-amdhsa-gfx950.s"))) as f:
        spacing.check(f.read())
    for name in os.listdir(obj_dir):
        if name.startswith((CHECKED + "-", CHECKED.replace(".hip", "-"))):
            os.remove(os.path.join(obj_dir, name))


def build_library(verbose: bool = True, jobs: int = 6) -> str:
    """Compile every translation unit and link the shared library.  Always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj_dir = os.path.join(PKG_DIR, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    procs, objs = [], []
    for src in SOURCES:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *HIPCC_FLAGS, "-I", INCLUDE, "-I", CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        if src == CHECKED:
            cmd.append("-save-temps=obj")
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            procs[0][1].wait()
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        lines = [l for l in out.splitlines() if "not a recognized feature for this target" not in l]
        if lines and verbose:
            print("\n".join(lines), flush=True)
        if p.returncode != 0:
            failed = True
            print(f"FAILED: {src}", file=sys.stderr)
    if failed:
        raise RuntimeError("hipcc failed")
    check_spacing(obj_dir)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB_PATH


if __name__ == "__main__":
    build_library()
