"""CPU: a device buffer whose allocation fails is empty.

The library grows its buffers when their size is too small, so a size kept from
a failed allocation would have the next call use a null pointer. The allocation
here is larger than any device (and fails as well where there is none).
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"

DRIVER = r"""
#include "runtime.h"
#include <cstdio>
int ddmgnn::fail(int code, const std::string&) { return code; }
int main() {
    ddmgnn::DevBuf<double> b;
    const hipError_t e = b.alloc((size_t)1 << 50);
    std::printf("%d %d %zu\n", e != hipSuccess, b.p == nullptr, b.n);
}
"""


@pytest.mark.skipif(not os.path.exists(f"{ROCM}/include/hip/hip_runtime.h"), reason="needs the ROCm headers")
def test_failed_allocation_leaves_an_empty_buffer(tmp_path):
    src, exe = tmp_path / "buffer.cpp", tmp_path / "buffer"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", f"{ROCM}/include",
                           "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_2402_08296_amd", "csrc"), str(src), "-o", str(exe),
                           "-L", f"{ROCM}/lib", "-lamdhip64", f"-Wl,-rpath,{ROCM}/lib"])
    assert subprocess.check_output([str(exe)], text=True).split() == ["1", "1", "0"]
