"""Builds libcalibatt.so (host pattern compiler + gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libcalibatt.so")
PROBE_PATH = os.path.join(PKG_DIR, "mfma_peak_probe.bin")  # stand-alone executable, see csrc/mfma_peak_probe.hip

SOURCES = ["compile_pattern.cpp", "anchor_map.cpp", "calibration.cpp", "skiplist.cpp", "split_plan.cpp", "sparse_attn_fwd.hip", "sparse_attn_split.hip"]

# Packed fp32 VALU forms are switched off for all device code.
HIP_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-Wno-inline-asm",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = True, extra_flags=()) -> str:
    import importlib.util
    import tempfile

    from concurrent.futures import ThreadPoolExecutor

    # One compilation per source, side by side.  --save-temps leaves the device assembly of this very compilation in its
    # working directory, which is checked for what the compiler does not guarantee: that the kernels that name registers
    # by hand keep them (csrc/check_named_regs.py), and that no MFMA result and no scalar register in a load's address is
    # read too early (csrc/check_mfma_waits.py, csrc/check_sgpr_waits.py).
    with tempfile.TemporaryDirectory() as tmp:
        def compile_one(source):
            stem = source.rsplit(".", 1)[0]
            work = os.path.join(tmp, stem)
            os.mkdir(work)
            obj = os.path.join(tmp, stem + ".o")
            cmd = [hipcc(), *[f for f in HIP_FLAGS if f != "-shared"], *extra_flags, "--save-temps", "-I",
                   os.path.join(ROOT, "include"), "-I", CSRC, "-c", os.path.join(CSRC, source), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True, cwd=work)
            return obj

        with ThreadPoolExecutor(len(SOURCES)) as pool:
            objects = list(pool.map(compile_one, SOURCES))
        subprocess.run([hipcc(), *HIP_FLAGS, *objects, "-o", LIB_PATH], check=True)
        texts = [open(os.path.join(tmp, s[:-4], s[:-4] + "-hip-amdgcn-amd-amdhsa-gfx950.s")).read()
                 for s in SOURCES if s.endswith(".hip")]
    for name in ("check_named_regs", "check_mfma_waits", "check_sgpr_waits"):
        spec = importlib.util.spec_from_file_location(name, os.path.join(CSRC, name + ".py"))
        mod = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(mod)
        problems = [p for text in texts for p in mod.check(text)]
        if problems:
            os.remove(LIB_PATH)
            raise RuntimeError(f"{name}.py rejects the compiled kernels:\n" + "\n".join(problems[:20]))
    probe = [hipcc(), *[f for f in HIP_FLAGS if f not in ("-fPIC", "-shared")], "-Wno-unused-value",
             os.path.join(CSRC, "mfma_peak_probe.hip"), "-o", PROBE_PATH]
    if verbose:
        print(" ".join(probe), flush=True)
    subprocess.run(probe, check=True)
    return LIB_PATH


if __name__ == "__main__":
    build(extra_flags=sys.argv[1:])
