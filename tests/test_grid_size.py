"""The grids of kernels that take one item a thread hold every item, beyond
2^28 of them too (explicit interpolation rows store 64 columns each, so 4.2
million rows are that many), and a count that no launch can hold is refused."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_04711_amd", "csrc")
SIZES = [0, 1, 255, 256, 257, 1 << 28, (1 << 28) + 1, 64 * 4194305, 2 * (1 << 31) - 512]
PROGRAM = """
#include "%s/cpm_internal.hpp"
namespace cpm { void set_error(const char*, ...) {} }
int main(int argc, char** argv) {
  for (int i = 1; i < argc; ++i) {
    const long long n = atoll(argv[i]);
    try { printf("%%d\\n", cpm::grid_for(n, 256)); }
    catch (const cpm::Error& e) { printf("refused %%d\\n", (int)(e.code == CPM_E_INVALID)); }
  }
}
"""


def test_a_grid_holds_every_item(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    include = "/opt/rocm/include"
    if not cxx or not os.path.isdir(include):
        pytest.skip("needs a C++ compiler and the HIP headers")
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text("#include <cstdlib>" + PROGRAM % CSRC)
    subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + include, str(src),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)] + [str(n) for n in SIZES + [1 << 32]], check=True,
                         capture_output=True, text=True).stdout.split("\n")
    for n, g in zip(SIZES, out):
        assert int(g) == max(1, -(-n // 256)), n
    assert out[len(SIZES)] == "refused 1"


def test_kernels_on_a_capped_grid_stride_over_it():
    sources = {f: open(os.path.join(CSRC, f)).read() for f in sorted(os.listdir(CSRC))
               if f.endswith(".hip")}
    capped = 0
    for f, text in sources.items():
        # a cap in the launch itself, or in a variable that the launch takes
        names = re.findall(r"const int (\w+) = grid_for\([^;]*, \d+, \d+\);", text)
        dims = [r"grid_for\([^()]*, \d+, \d+\)"] + [r"%s\b" % n for n in set(names)]
        for m in re.finditer(r"hipLaunchKernelGGL\(\(?(k_\w+)[^;]*?dim3\((?:%s)\)" % "|".join(dims),
                             text):
            kernel = m.group(1)
            body = text[re.search(r"__global__[^;{]*\b%s\(" % kernel, text).start():]
            body = body[:body.index("\n}\n")]
            assert "gridDim.x" in body, (f, kernel)
            capped += 1
    assert capped >= 5
