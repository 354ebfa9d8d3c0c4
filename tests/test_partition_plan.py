"""The overlap partition's scratch, for every number of points (host arithmetic, no GPU): the kernels' parts lie within the bytes that
callers are told to bring, and the two-launch form's chunks, counters and edges within what its kernels hold."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdio.h>
#include "dw.h"
#include "dw_partition_plan.h"
int main() {
  for (int64_t n = 1; n <= DW_MAX_POINTS; ++n) {
    const dw::PartitionPlan p = dw::partition_plan(n);
    const int64_t points = (int64_t)dw::kChunkThreads * p.per;
    const bool chunks = p.chunks == 0 || (p.chunks <= dw::kMaxChunks && p.chunks * points >= n && (p.chunks - 1) * points < n &&
                                          points <= 65535 && p.nb * 4 <= 32768);
    if (p.bytes > dw::partition_scratch_bytes(n) || p.nb != 1 << p.bits || !chunks) { printf("n = %lld\n", (long long)n); return 1; }
  }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")
def test_every_set_fits_its_scratch(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2409_09242_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
