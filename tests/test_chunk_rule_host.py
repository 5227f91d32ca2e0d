"""The rule that cuts a sample into chunks, compiled from the library's header
for the host: the rows set aside for samples of up to n events hold the rows of
every one of them, also where the largest chunk leaves more workgroups than the
rule aims at (beyond 2^22 events per workgroup)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1710_08826_amd", "csrc")
PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#define __host__
#define __device__
#define __HIPCC_RTC__
namespace __hip_internal { using ::int32_t; using ::int64_t; using ::uint32_t; using ::uint64_t; }
#include "model.hpp"
int main() {
  const fn::ChunkRule rules[] = {{1024, 2048}, {256, 512}, {256, 2}, {1024, 0}, {4096, 0}, {fn::kMaxChunk, 3}};
  long long bad = 0, seen = 0;
  for (const auto& r : rules) {
    const int64_t slots = r.slots > 0 ? r.slots : 64;
    const int64_t marks[] = {1, 255, 1000, (int64_t)r.lo * slots, 3 * (int64_t)r.lo * slots + 7,
                             (int64_t)fn::kMaxChunk * slots, (int64_t)fn::kMaxChunk * slots * 5 / 4};
    for (int64_t n : marks)
      for (int64_t d = -700; d <= 700; d += 7) {
        const int64_t most = n + d;
        if (most < 1) continue;
        const int64_t rows = r.rows_upto(most);
        // every size near the top, and a spread of smaller ones
        for (int64_t k = 0; k < 400; ++k) {
          const int64_t m = k < 200 ? most - 3 * k : most - (most / 200) * (k - 200);
          if (m < 1) continue;
          const int64_t c = r(m), need = (m + c - 1) / c;
          ++seen;
          if (need > rows) ++bad;
          if (c % fn::kBlock || c > fn::kMaxChunk) ++bad;
        }
        // and not more than the largest count of chunks of any size needs
        if (r.slots > 0 && most <= (int64_t)fn::kMaxChunk * r.slots && rows > r.slots) ++bad;
      }
  }
  std::printf("%lld %lld\n", bad, seen);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_rows_of_every_sample_fit(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    bad, seen = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert seen > 100_000 and bad == 0
