"""Build the C-ABI library ``libpreserve.so`` for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys
import sysconfig
from typing import List

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpreserve.so")

MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["api.hip", "model_file.cpp", "rowops.hip", "encoder_f32.hip", "encoder_bf16.hip", "gemm_bf16.hip", "skinny_gemm.hip", "small_gemm.hip", "attention_bf16.hip",
           "anticipate.hip", "lookahead.hip", "scaler.hip", "router.hip", "forecaster.hip", "stream_read.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",

         "-I", INCLUDE, "-I", CSRC]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


# Per-file additions.  attention: MFMA results go straight to ordinary VGPRs, since the softmax reads
# every one of them with VALU instructions (the default sends them through the accumulation registers).
EXTRA_FLAGS = {"attention_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    if src.endswith(".cpp"):       # host-only code: the plain host compiler
        cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-I", INCLUDE, "-I", CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
    else:
        cmd = [_hipcc(), *FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def _build_marshal() -> None:
    """The binding's argument marshalling as an extension module (host code, torch's headers)."""
    import torch
    from torch.utils import cpp_extension
    tmp = MARSHAL + f".tmp{os.getpid()}"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", INCLUDE, "-I", sysconfig.get_paths()["include"]]
    for p in cpp_extension.include_paths():
        cmd += ["-isystem", p]
    cmd.append(os.path.join(CSRC, "marshal.cpp"))
    for p in cpp_extension.library_paths():
        cmd += ["-L", p]
    r = subprocess.run(cmd + ["-ltorch_python", "-ltorch_cpu", "-lc10", "-o", tmp], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for marshal.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, MARSHAL)


def build_library(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        marshal = ex.submit(_build_marshal)
        objs: List[str] = list(ex.map(_compile, SOURCES))
        marshal.result()
    tmp = LIB + f".tmp{os.getpid()}"
    r = subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build_library()
