"""Builds liblightkv.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "liblightkv.so")
PROBE_LIB_PATH = os.path.join(HERE, "liblightkv_probe.so")   # measurement kernels for bench.py --pass ceilings, nothing of the method
SOURCES = ["lk_api.hip", "lk_windows.hip", "lk_score_fd.hip", "lk_score_fd_big.hip", "lk_fd_dump.hip", "lk_score_xi.hip", "lk_xi_seq.hip", "lk_select.hip", "lk_select_edges.hip", "lk_select_pair.hip", "lk_rows.hip", "lk_fused.hip", "lk_schedule.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed-fp32 instruction forms are kept out of the generated code on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# matrix-core results that vector instructions go on with at once: left alone the compiler puts them into accumulation
# registers and copies every one of them out (16 copies per 32 x 32 tile)
FILE_FLAGS = {src: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
              for src in ("lk_score_xi.hip", "lk_fused.hip")}


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: the HIP toolchain is required to build liblightkv.so")
    return exe


def build(verbose: bool = True, jobs: int = 6) -> str:
    hipcc = _hipcc()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, *FILE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB_PATH + ".tmp"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB_PATH)
    if verbose:
        print("built", LIB_PATH)
    probe_obj = compile_one("lk_probe.hip")
    tmp = PROBE_LIB_PATH + ".tmp"
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, probe_obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, PROBE_LIB_PATH)
    if verbose:
        print("built", PROBE_LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build()
