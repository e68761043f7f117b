"""GPU: daf_linear on either side of the rule that picks its 128 x 128 kernel
(small_tiles_pay in gemm.h), against the CPU oracle, and the rule itself at these
sizes. Bars as in test_gpu_linear_tiles.py: half a bf16 ulp and fp32 sums."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from conftest import ROOT

SMALL = [(1, 128, 64), (63, 384, 1024), (64, 2304, 1088), (127, 128, 192), (128, 640, 1536), (129, 256, 1472),
         (512, 128, 960), (257, 1024, 320), (1000, 2048, 512), (513, 4096, 256), (4097, 512, 512)]
LARGE = [(63, 2176, 1088), (1, 128, 1152), (128, 384, 1600), (129, 256, 2112), (255, 128, 4160), (256, 640, 1600),
         (513, 640, 2112), (640, 768, 2112), (641, 640, 4160), (767, 640, 4160), (1025, 4096, 576), (1025, 8192, 512),
         (2049, 2048, 576), (5000, 3328, 64),
         (5134, 2048, 1088)]  # 20 x 8 tiles, more than half a round: every tile whole, 14 last rows


def test_rule(tmp_path):
    with open(os.path.join(ROOT, "paper_2607_21599_amd", "csrc", "gemm.h")) as f:
        rule = re.search(r"constexpr bool small_tiles_pay\(.*?\n}\n", f.read(), re.S).group(0)
    body = "".join(f"if (small_tiles_pay({m}, {n}, {k}) != {int(s)}) return {i + 1};\n"
                   for i, (m, n, k, s) in enumerate([(*x, True) for x in SMALL] + [(*x, False) for x in LARGE]))
    (tmp_path / "r.cpp").write_text("#include <cstdint>\n" + rule + "int main() {\n" + body + "}\n")
    subprocess.run(["g++", "-std=c++17", str(tmp_path / "r.cpp"), "-o", str(tmp_path / "r")], check=True)
    assert subprocess.run([str(tmp_path / "r")]).returncode == 0


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SMALL + LARGE)
def test_linear_both_kernels(M, N, K):
    import torch

    import daf_inputs as di
    import paper_2607_21599_amd as daf
    from oracle import decoder as dec
    from test_gpu_linear_tiles import _check, _dev
    w = di.raw_to_f32
    A, W, b, R = di.make_linear_case(M, N, K, seed=M + N + K, bias=True, residual=True)
    full = dec.linear(w(A), w(W))
    for bias, res in ((False, False), (True, True)):
        C = torch.full((M + 3, N), 7.0, dtype=torch.bfloat16, device="cuda")
        if res:
            C[:M] = _dev(R)
        daf.daf_linear(M, N, K, _dev(A), _dev(W), _dev(b) if bias else None, C if res else None, C)
        torch.cuda.synchronize()
        _check(C[:M], full + w(b)[None, :] + w(R) if bias else full, f"linear {M}x{N}x{K}")
        assert torch.all(C[M:] == 7.0), "rows past M were written"
