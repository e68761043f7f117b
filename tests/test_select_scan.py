"""CPU: the top-n kernel's scan over its waves, compiled here from select.hip with
the undefined-behaviour sanitizer. It adds two counts packed in one word, which for
a full slab of keys above the threshold reach 2^31."""
from __future__ import annotations

import os
import re
import subprocess

from conftest import ROOT

MAIN = r"""
#include <cstdio>
#include <initializer_list>
#define __device__
#define __forceinline__ inline
#define __syncthreads()
static struct { unsigned x; } threadIdx;
constexpr int kTopnWaves = 16;
%s
int main() {
  for (unsigned gt : {2048u, 2047u, 0u}) {  // keys above the threshold per wave, the rest equal to it
    const unsigned v = gt << 16 | (2048u - gt);
    for (unsigned w = 0; w < 16; ++w) {
      SCAN_T wsum[kTopnWaves], sum;
      for (auto &x : wsum) x = v;
      threadIdx.x = 64 * w;
      const unsigned before = wave_scan(v, wsum, sum), total = sum;
      if (before >> 16 != w * gt || (before & 0xffffu) != w * (2048u - gt)) return 1;
      if (total >> 16 != 16 * gt || (total & 0xffffu) != 16 * (2048u - gt)) return 2;
    }
  }
  puts("ok");
}
"""


def test_packed_counts_of_a_full_slab(tmp_path):
    with open(os.path.join(ROOT, "paper_2607_21599_amd", "csrc", "select.hip")) as f:
        src = f.read()
    fn = re.search(r"__device__ __forceinline__ (\w+) wave_scan\(.*?\n}\n", src, re.S)
    cpp = tmp_path / "scan.cpp"
    cpp.write_text((MAIN % fn.group(0)).replace("SCAN_T", fn.group(1)))
    exe = tmp_path / "scan"
    subprocess.run(["g++", "-std=c++17", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all", str(cpp), "-o",
                    str(exe)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True)
    assert got.returncode == 0 and got.stdout == "ok\n", got.stderr
