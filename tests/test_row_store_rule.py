"""The rule by which a GEMM tile's outputs leave in streaming or in plain stores (RowStore::streams), compiled for the host and
called on either side of its lines: alignment of every row, K, the outputs' own bytes whatever the stride of the buffer
they are a slice of.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "row_store.hpp"
int main(int argc, char** argv) {
  for (int i = 1; i + 5 < argc; i += 6) {
    const auto n = [&](int j) { return atoll(argv[i + j]); };
    const void* Y = reinterpret_cast<const void*>(n(1));
    const bool s = n(0) ? wush::RowStore<true, 2>::streams(Y, n(2), (int)n(3), (int)n(4), (int)n(5))
                        : wush::RowStore<false, 2>::streams(Y, n(2), (int)n(3), (int)n(4), (int)n(5));
    printf("%d", s);
  }
  return 0;
}
"""

# (FP32 output, address of Y, row stride, tokens, channels, K) -> streaming
CASES = [((0, 4096, 1024, 64, 1024, 256), 1),          # BF16 rows at multiples of 64 bytes: at any K
         ((0, 4096 + 32, 1024, 64, 1024, 256), 0),     # the first row off them
         ((0, 4096, 1000, 64, 1000, 4064), 0), ((0, 4096, 1000, 64, 1000, 4096), 1),       # rows at multiples of 16 bytes
         ((0, 4096, 1001, 64, 1001, 4096), 0), ((0, 4096, 1001, 64, 1001, 8160), 0), ((0, 4096, 1001, 64, 1001, 8192), 1),
         ((1, 4096, 1001, 64, 1001, 8160), 0), ((1, 4096, 1001, 64, 1001, 8192), 1),
         ((1, 4096, 1001, 1047, 1001, 256), 0), ((1, 4096, 1001, 1048, 1001, 256), 1),     # FP32: above 4 MiB ...
         ((1, 4096, 1001, 4190, 1001, 256), 1), ((1, 4096, 1001, 4191, 1001, 256), 0),     # ... up to 16 MiB
         ((1, 4096, 4003, 1047, 1001, 256), 0), ((1, 4096, 4003, 4190, 1001, 256), 1),     # a slice of a wider buffer: the same
         ((0, 4096, 1001, 4190, 1001, 256), 0), ((0, 4096, 1001, 8000, 1001, 256), 0)]     # no such range for BF16


def test_streams(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "rule.hip", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2512_00956_amd", "csrc"), str(src), "-o", str(exe)], check=True, capture_output=True)
    args = [str(v) for case, _ in CASES for v in case]
    out = subprocess.run([str(exe), *args], check=True, capture_output=True, text=True).stdout
    assert out == "".join(str(want) for _, want in CASES)
