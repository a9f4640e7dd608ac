"""Registers of compiled kernels, from the built library's own metadata (no GPU): loops over slabs whose values stay alive by mistake show
as registers that go to memory and back, which no result shows."""
import os
import re
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2302_12510_amd import build

LLVM = "/opt/rocm/llvm/bin/"
TARGET = "hipv4-amdgcn-amd-amdhsa--gfx950"


def run(*cmd):
    return subprocess.run(cmd, check=True, capture_output=True, text=True).stdout


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{mangled name of a kernel: vector registers that are spilled}"""
    if not all(os.path.exists(p) for p in (build.LIB, LLVM + "clang-offload-bundler", LLVM + "llvm-objcopy", LLVM + "llvm-readelf")):
        pytest.skip("needs the built library and the compiler's tools")
    d = str(tmp_path_factory.mktemp("kernels"))
    run(LLVM + "llvm-objcopy", "--dump-section", f".hip_fatbin={d}/all", build.LIB, "/dev/null")
    data = open(f"{d}/all", "rb").read()
    bundles, at = [], data.find(b"CCOB")
    while at >= 0:                                       # compressed bundles, one per source: magic, version, method, size of all
        version, = struct.unpack_from("<H", data, at + 4)
        size, = struct.unpack_from("<Q" if version >= 3 else "<I", data, at + 8)
        bundles.append(data[at:at + size])
        at = data.find(b"CCOB", at + size)

    def notes(i):
        name = f"{d}/{i}"
        with open(name, "wb") as f:
            f.write(bundles[i])
        run(LLVM + "clang-offload-bundler", "--type=o", "--unbundle", f"--targets={TARGET}", f"--input={name}", f"--output={name}.elf")
        text = run(LLVM + "llvm-readelf", "--notes", name + ".elf")
        os.remove(name + ".elf")
        return re.findall(r"\.name: +(\S+)\n(?:.*\n)*?.*\.vgpr_spill_count: +(\d+)", text)
    found = {}
    with ThreadPoolExecutor(4) as ex:
        for pairs in ex.map(notes, range(len(bundles))):
            for name, count in pairs:
                found[name] = int(count)
    return found


def test_weight_stationary_fp32(spills):
    """Template arguments: formats of A and W, convolution (0: product), blocks of 32 columns, outputs (0: fp32).  What the accumulators, two K
    steps of codes and the epilogue need is 6 to 12 registers more than four waves per SIMD have, for a convolution up to 33."""
    kernels = {tuple(map(int, re.findall(r"Li(\d+)E", name))): n for name, n in spills.items() if "14gemm_ws_kernelI" in name}
    kernels = {a: n for a, n in kernels.items() if a[4] == 0}
    assert len(kernels) == 8 * 4 * 3 * 2
    assert {a: n for a, n in kernels.items() if n > (0 if a[3] == 4 else 12 if a[2] == 0 else 33)} == {}
