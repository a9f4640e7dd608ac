"""Builds libdybit.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdybit.so")
NATIVE = os.path.join(HERE, "_native.so")         # the binding's argument marshalling (needs torch's headers)
# (source, object stem, extra flags): the tiled kernels are compiled once per weight format
SOURCES = [
    ("host.cpp", "host", []),
    ("quantize.hip", "quantize", []),
    ("metric.hip", "metric", []),
    ("dwconv.hip", "dwconv", []),
    ("pool.hip", "pool", []),
    ("search.cpp", "search", []),
    ("gemm.hip", "gemm", []),
    ("gemm_dispatch.cpp", "gemm_dispatch", []),
    ("gemm_six.hip", "gemm_six", []),
    ("gemm_fast.hip", "gemm_fast_w4", ["-DDYBIT_FAST_W=0"]),
    ("gemm_fast.hip", "gemm_fast_w8", ["-DDYBIT_FAST_W=2"]),
    ("gemm_fast.hip", "gemm_fast_w6", ["-DDYBIT_FAST_W=4"]),
    ("gemm_fast.hip", "gemm_fast_w2", ["-DDYBIT_FAST_W=6"]),
    ("gemm_mid.hip", "gemm_mid_w4", ["-DDYBIT_MID_W=0"]),
    ("gemm_mid.hip", "gemm_mid_w8", ["-DDYBIT_MID_W=2"]),
    ("gemm_mid.hip", "gemm_mid_w6", ["-DDYBIT_MID_W=4"]),
    ("gemm_mid.hip", "gemm_mid_w2", ["-DDYBIT_MID_W=6"]),
    ("gemm_f8.hip", "gemm_f8_w4", ["-DDYBIT_F8_W=0"]),
    ("gemm_f8.hip", "gemm_f8_w2", ["-DDYBIT_F8_W=6"]),
    ("gemm_ws.hip", "gemm_ws_w4", ["-DDYBIT_WS_W=0"]),
    ("gemm_ws.hip", "gemm_ws_w8", ["-DDYBIT_WS_W=2"]),
    ("gemm_ws.hip", "gemm_ws_w6", ["-DDYBIT_WS_W=4"]),
    ("gemm_ws.hip", "gemm_ws_w2", ["-DDYBIT_WS_W=6"]),
    ("gemm_small.hip", "gemm_small_w4", ["-DDYBIT_SMALL_W=0"]),
    ("gemm_small.hip", "gemm_small_w4_wb", ["-DDYBIT_SMALL_W=0", "-DDYBIT_WB=1"]),
    ("gemm_small.hip", "gemm_small_w8", ["-DDYBIT_SMALL_W=2"]),
    ("gemm_small.hip", "gemm_small_w8_wb", ["-DDYBIT_SMALL_W=2", "-DDYBIT_WB=1"]),
    ("gemm_small.hip", "gemm_small_w6", ["-DDYBIT_SMALL_W=4"]),
    ("gemm_small.hip", "gemm_small_w6_wb", ["-DDYBIT_SMALL_W=4", "-DDYBIT_WB=1"]),
    ("gemm_small.hip", "gemm_small_w2", ["-DDYBIT_SMALL_W=6"]),
    ("gemm_small.hip", "gemm_small_w2_wb", ["-DDYBIT_SMALL_W=6", "-DDYBIT_WB=1"]),
    ("gemm_group.hip", "gemm_group_w4", ["-DDYBIT_GROUP_W=0"]),
    ("gemm_group.hip", "gemm_group_w8", ["-DDYBIT_GROUP_W=2"]),
    ("gemm_group.hip", "gemm_group_w6", ["-DDYBIT_GROUP_W=4"]),
    ("gemm_group.hip", "gemm_group_w2", ["-DDYBIT_GROUP_W=6"]),
    # write-back builds of the same kernels (epilogue also encodes the results as DyBit codes)
    ("gemm.hip", "gemm_wb_a2", ["-DDYBIT_WB=1", "-DDYBIT_GEN_A=2"]),
    ("gemm.hip", "gemm_wb_a4", ["-DDYBIT_WB=1", "-DDYBIT_GEN_A=4"]),
    ("gemm.hip", "gemm_wb_a6", ["-DDYBIT_WB=1", "-DDYBIT_GEN_A=6"]),
    ("gemm.hip", "gemm_wb_a8", ["-DDYBIT_WB=1", "-DDYBIT_GEN_A=8"]),
    ("gemm_fast.hip", "gemm_fast_w4_wb", ["-DDYBIT_FAST_W=0", "-DDYBIT_WB=1"]),
    ("gemm_fast.hip", "gemm_fast_w8_wb", ["-DDYBIT_FAST_W=2", "-DDYBIT_WB=1"]),
    ("gemm_fast.hip", "gemm_fast_w6_wb", ["-DDYBIT_FAST_W=4", "-DDYBIT_WB=1"]),
    ("gemm_fast.hip", "gemm_fast_w2_wb", ["-DDYBIT_FAST_W=6", "-DDYBIT_WB=1"]),
    ("gemm_mid.hip", "gemm_mid_w4_wb", ["-DDYBIT_MID_W=0", "-DDYBIT_WB=1"]),
    ("gemm_mid.hip", "gemm_mid_w8_wb", ["-DDYBIT_MID_W=2", "-DDYBIT_WB=1"]),
    ("gemm_mid.hip", "gemm_mid_w6_wb", ["-DDYBIT_MID_W=4", "-DDYBIT_WB=1"]),
    ("gemm_mid.hip", "gemm_mid_w2_wb", ["-DDYBIT_MID_W=6", "-DDYBIT_WB=1"]),
    ("gemm_f8.hip", "gemm_f8_w4_wb", ["-DDYBIT_F8_W=0", "-DDYBIT_WB=1"]),
    ("gemm_f8.hip", "gemm_f8_w2_wb", ["-DDYBIT_F8_W=6", "-DDYBIT_WB=1"]),
    ("gemm_ws.hip", "gemm_ws_w4_wb", ["-DDYBIT_WS_W=0", "-DDYBIT_WB=1"]),
    ("gemm_ws.hip", "gemm_ws_w8_wb", ["-DDYBIT_WS_W=2", "-DDYBIT_WB=1"]),
    ("gemm_ws.hip", "gemm_ws_w6_wb", ["-DDYBIT_WS_W=4", "-DDYBIT_WB=1"]),
    ("gemm_ws.hip", "gemm_ws_w2_wb", ["-DDYBIT_WS_W=6", "-DDYBIT_WB=1"]),
    # codes-only builds (no fp32 output: epilogue on the transposed product)
    ("gemm_mid.hip", "gemm_mid_w4_co", ["-DDYBIT_MID_W=0", "-DDYBIT_WB=2"]),
    ("gemm_mid.hip", "gemm_mid_w8_co", ["-DDYBIT_MID_W=2", "-DDYBIT_WB=2"]),
    ("gemm_mid.hip", "gemm_mid_w6_co", ["-DDYBIT_MID_W=4", "-DDYBIT_WB=2"]),
    ("gemm_mid.hip", "gemm_mid_w2_co", ["-DDYBIT_MID_W=6", "-DDYBIT_WB=2"]),
    ("gemm_f8.hip", "gemm_f8_w4_co", ["-DDYBIT_F8_W=0", "-DDYBIT_WB=2"]),
    ("gemm_f8.hip", "gemm_f8_w2_co", ["-DDYBIT_F8_W=6", "-DDYBIT_WB=2"]),
    ("gemm_ws.hip", "gemm_ws_w4_co", ["-DDYBIT_WS_W=0", "-DDYBIT_WB=2"]),
    ("gemm_ws.hip", "gemm_ws_w8_co", ["-DDYBIT_WS_W=2", "-DDYBIT_WB=2"]),
    ("gemm_ws.hip", "gemm_ws_w6_co", ["-DDYBIT_WS_W=4", "-DDYBIT_WB=2"]),
    ("gemm_ws.hip", "gemm_ws_w2_co", ["-DDYBIT_WS_W=6", "-DDYBIT_WB=2"]),
    ("conv_few.hip", "conv_few_w4", ["-DDYBIT_FEW_W=0"]),
    ("conv_few.hip", "conv_few_w4_co", ["-DDYBIT_FEW_W=0", "-DDYBIT_WB=2"]),
    ("conv_few.hip", "conv_few_w8", ["-DDYBIT_FEW_W=2"]),
    ("conv_few.hip", "conv_few_w8_co", ["-DDYBIT_FEW_W=2", "-DDYBIT_WB=2"]),
    ("conv_few.hip", "conv_few_w6", ["-DDYBIT_FEW_W=4"]),
    ("conv_few.hip", "conv_few_w6_co", ["-DDYBIT_FEW_W=4", "-DDYBIT_WB=2"]),
    ("conv_few.hip", "conv_few_w2", ["-DDYBIT_FEW_W=6"]),
    ("conv_few.hip", "conv_few_w2_co", ["-DDYBIT_FEW_W=6", "-DDYBIT_WB=2"]),
    ("conv_patch.hip", "conv_patch_w4", ["-DDYBIT_PATCH_W=0"]),
    ("conv_patch.hip", "conv_patch_w4_wb", ["-DDYBIT_PATCH_W=0", "-DDYBIT_WB=1"]),
    ("conv_patch.hip", "conv_patch_w4_co", ["-DDYBIT_PATCH_W=0", "-DDYBIT_WB=2"]),
    ("conv_patch.hip", "conv_patch_w8", ["-DDYBIT_PATCH_W=2"]),
    ("conv_patch.hip", "conv_patch_w8_wb", ["-DDYBIT_PATCH_W=2", "-DDYBIT_WB=1"]),
    ("conv_patch.hip", "conv_patch_w8_co", ["-DDYBIT_PATCH_W=2", "-DDYBIT_WB=2"]),
    ("conv_patch.hip", "conv_patch_w6", ["-DDYBIT_PATCH_W=4"]),
    ("conv_patch.hip", "conv_patch_w6_wb", ["-DDYBIT_PATCH_W=4", "-DDYBIT_WB=1"]),
    ("conv_patch.hip", "conv_patch_w6_co", ["-DDYBIT_PATCH_W=4", "-DDYBIT_WB=2"]),
    ("conv_patch.hip", "conv_patch_w2", ["-DDYBIT_PATCH_W=6"]),
    ("conv_patch.hip", "conv_patch_w2_wb", ["-DDYBIT_PATCH_W=6", "-DDYBIT_WB=1"]),
    ("conv_patch.hip", "conv_patch_w2_co", ["-DDYBIT_PATCH_W=6", "-DDYBIT_WB=2"]),
    ("diag.hip", "diag", []),
]
FLAGS = ["--offload-arch=gfx950", "--offload-compress", "-O3", "-fPIC", "-std=c++17",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(item) -> str:
    src, stem, extra = item
    obj = os.path.join(CSRC, stem + ".o")
    cmd = [_hipcc(), *FLAGS, *extra, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in p.stderr.splitlines() if "not a recognized feature" not in l)
    if p.returncode:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        print(err)
    return obj


# Longest compilations first, so that the pool's last jobs are short ones.
_ORDER = ("gemm", "gemm_wb", "gemm_mid", "gemm_ws", "gemm_f8", "gemm_fast", "conv_few", "gemm_small", "quantize")


def _rank(item) -> int:
    stem = item[1]
    for i, prefix in enumerate(_ORDER):
        if stem == prefix or (i >= 1 and stem.startswith(prefix)):
            return i
    return len(_ORDER)


def _build_native() -> None:
    spec = importlib.util.find_spec("torch")
    torch_dir = spec.submodule_search_locations[0]
    inc, libs = os.path.join(torch_dir, "include"), os.path.join(torch_dir, "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f"-I{inc}", f"-I{inc}/torch/csrc/api/include", "-I/opt/rocm/include", f"-I{sysconfig.get_paths()['include']}",
           os.path.join(CSRC, "binding_native.cpp"), "-o", NATIVE, f"-L{HERE}", "-l:libdybit.so",
           f"-L{libs}", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode:
        raise RuntimeError("g++ failed on binding_native.cpp:\n" + p.stderr)


def build(verbose: bool = True) -> str:
    jobs = sorted(SOURCES, key=_rank)
    with ThreadPoolExecutor(max_workers=min(len(jobs), os.cpu_count() or 8)) as ex:
        objs = list(ex.map(_compile, jobs))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode:
        raise RuntimeError("link failed:\n" + p.stderr)
    _build_native()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
