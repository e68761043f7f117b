"""CPU: which tiles of a projection run whole, as halves or in k pieces. The plan
is compiled here from gemm.hip by itself; the decoder-layer tests of
test_gpu_layer.py and test_gpu_layer_pieces.py name these plans as what they run."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2607_21599_amd", "csrc")
H, I, QW, KW = 3584, 18944, 3584, 512  # Qwen2.5-7B widths
PROJ = {"qkv": (H, (QW, KW, KW), 0), "o": (QW, (H,), 0), "gu": (H, (I,), 1), "down": (I, (H,), 0)}
MAIN = """
#include <cstdio>
#include <cstdlib>
#include <cstddef>
#include <cstdint>
#include <algorithm>
#include "gemm.h"
namespace daf {
constexpr int kTK = 64, kCus = 256;
%s
%s
}
int main(int c, char **a) {
  daf::GemmPlan p{};
  p.j.M = atol(a[1]), p.j.K = atoi(a[2]), p.j.glu = atoi(a[3]), p.part = atoi(a[4]) ? (float *)64 : nullptr;
  for (int i = 5; i < c; ++i) p.j.seg[p.j.n_segs++].N = atoi(a[i]);
  daf::plan_job(p, daf::kGemmPieceBytes);
  printf("%%d %%d %%d %%d", p.n_full, p.n_cut, p.n_half - 2 * p.n_cut, p.k_parts);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    (tmp / "hip").mkdir()
    (tmp / "hip" / "hip_runtime.h").write_text("typedef int hipError_t;\ntypedef void *hipStream_t;\n")
    with open(os.path.join(CSRC, "gemm.hip")) as f:
        src = f.read()
    assert "constexpr int kTK = 64;" in src and "constexpr int kCus = 256;" in src
    struct = re.search(r"struct GemmPlan \{.*?\n};\n", src, re.S).group(0)
    fn = re.search(r"void plan_job\(.*?\n}\n", src, re.S).group(0)
    (tmp / "plan.cpp").write_text(MAIN % (struct, fn))
    subprocess.run(["g++", "-std=c++17", f"-I{tmp}", f"-I{CSRC}", str(tmp / "plan.cpp"), "-o", str(tmp / "plan")],
                   check=True)

    def run(rows, proj):
        """(whole 256-row tiles, tiles cut in halves, 128-row units of the last rows, pieces along k)"""
        K, ns, glu = PROJ[proj]
        out = subprocess.run([str(tmp / "plan"), str(rows), str(K), str(glu), str(int(not glu))] + [str(n) for n in ns],
                             check=True, capture_output=True, text=True).stdout
        return tuple(int(x) for x in out.split())
    return run


@pytest.mark.parametrize("rows,proj,want", [
    # test_gpu_layer.py
    (986, "qkv", (0, 72, 0, 1)), (986, "o", (0, 56, 0, 2)), (986, "gu", (512, 80, 0, 1)), (986, "down", (0, 56, 0, 2)),
    (2586, "qkv", (180, 0, 18, 1)), (2586, "gu", (1480, 0, 148, 1)), (2586, "down", (140, 0, 14, 1)),
    (9300, "qkv", (648, 0, 18, 1)), (9300, "o", (504, 0, 14, 1)), (9300, "down", (504, 0, 14, 1)),
    # test_gpu_layer_pieces.py
    (100, "qkv", (0, 0, 18, 8)), (100, "o", (0, 0, 14, 9)), (100, "down", (0, 0, 14, 18)),
    (300, "qkv", (0, 18, 18, 4)), (300, "o", (0, 14, 14, 5)), (300, "down", (0, 14, 14, 6)),
    (500, "qkv", (0, 36, 0, 3)), (500, "o", (0, 28, 0, 4)), (500, "down", (0, 28, 0, 4)),
    (640, "qkv", (0, 36, 18, 2)), (640, "o", (0, 28, 14, 3)), (640, "gu", (256, 40, 148, 1)),
    (5134, "qkv", (256, 104, 18, 1)), (5134, "o", (256, 24, 14, 4)), (5134, "down", (256, 24, 14, 4))])
def test_plans_that_the_layer_tests_run(plan, rows, proj, want):
    assert plan(rows, proj) == want
