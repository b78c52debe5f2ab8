"""The library's host threads: what a share throws reaches the caller (it would end the program
otherwise), after every share has ended."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include "pdmi_host.h"
int main()
{
    std::atomic<int64_t> done{0};
    try {
        pdmi::host::parallel_for(100000, [&](int64_t lo, int64_t hi) {
            if (lo > 0) throw std::bad_alloc();
            done += hi - lo;
        });
    } catch (const std::bad_alloc&) {
        int64_t sum = 0;
        std::mutex mu;
        pdmi::host::parallel_for(100000, [&](int64_t lo, int64_t hi) {
            std::lock_guard<std::mutex> lock(mu);
            sum += hi - lo;
        });
        return done > 0 && sum == 100000 ? 0 : 2;
    }
    return pdmi::host::n_threads() > 1 ? 1 : 0;
}
'''


def test_exceptions_leave_the_threads(tmp_path):
    src = tmp_path / "threads.cpp"
    src.write_text("#include <mutex>\n" + PROGRAM)
    exe = tmp_path / "threads"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2105_04150_amd", "csrc"),
                    str(src), "-o", str(exe), "-pthread"], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
