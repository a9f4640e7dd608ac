"""dybit_set_option from one thread while another calls: the kernel of a call follows from one reading of the options.  The program launches nothing
(its own launch functions are found before the runtime's), so its made-up pointers go nowhere."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <thread>
#include "dybit.h"
struct Dim { unsigned x, y, z; };
extern "C" int hipFuncSetAttribute(const void *, int, int) { return 0; }
extern "C" int __hipPushCallConfiguration(Dim, Dim, size_t, void *) { return 1; }        // not 0: the launch is left out
extern "C" int hipGetLastError() { return 0; }
int main()
{
    std::atomic<bool> done{false};
    std::thread other([&] { while (!done) { dybit_set_option("gemm_mfma", "f16"); dybit_set_option("gemm_mfma", "auto"); } });
    uint8_t *const p = (uint8_t *)0x10000;
    const dybit_fmt a{8, 1}, w{4, 1};
    long six = 0, others = 0;
    // both answers, many times each: a second reading of the options within a call would soon meet another answer than the first
    for (long calls = 0; calls < 4000000 && (calls < 1000000 || six < 1000 || others < 1000); ++calls) {
        dybit_gemm_work(8192, 8192, 8192, p, a, (float *)p, p, w, (float *)p, nullptr, 0, (float *)p, 8192, p, (size_t)1 << 31, nullptr);
        const int k = dybit_last_gemm_kernel();
        k == DYBIT_KERNEL_F6_256 ? ++six : ++others;
        if (k != DYBIT_KERNEL_F6_256 && k != DYBIT_KERNEL_F16_256) return 2;
    }
    done = true;
    other.join();
    std::printf("%ld %ld\n", six, others);
}
"""


def test_split_product_while_options_change(tmp_path):
    (tmp_path / "program.cpp").write_text(PROGRAM)
    package = os.path.join(ROOT, "paper_2302_12510_amd")
    program = str(tmp_path / "program")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", f"-I{ROOT}/include", str(tmp_path / "program.cpp"), "-o", program, "-rdynamic",
                    f"-L{package}", "-l:libdybit.so", f"-Wl,-rpath,{package}", "-Wl,-rpath-link,/opt/rocm/lib"], check=True)
    p = subprocess.run([program], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, (p.returncode, p.stdout, p.stderr)
    six, others = map(int, p.stdout.split())
    assert six >= 1000 and others >= 1000
