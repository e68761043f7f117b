"""CPU: which launches of causal attention take 64-row blocks. The rule's header
is compiled here by itself; the points are times with 64 rows over times with
128, measured with rows at the end of a key sequence (mean chain of key tiles
over the longest: 0.5 for a triangle, towards 1 for long keys)."""
from __future__ import annotations

import os
import subprocess

from conftest import ROOT

SHARES = (0.50, 0.57, 0.63, 0.69, 0.75, 0.83, 0.92)
MEASURED = {
    (128, 56): (0.76, 0.72, 0.72, 0.71, 0.72, 0.72, 0.73),
    (128, 140): (0.76, 0.77, 0.76, 0.77, 0.77, 0.78, 0.84),
    (128, 196): (0.78, 0.78, 0.78, 0.78, 0.79, 0.81, 0.88),
    (128, 252): (0.74, 0.73, 0.75, 0.76, 0.77, 0.81, 0.79),
    (128, 280): (0.76, 0.75, 0.77, 0.89, 1.02, 1.25, 1.18),
    (128, 336): (0.76, 0.87, 0.97, 1.09, 1.21, 1.24, 1.17),
    (128, 392): (0.87, 0.97, 1.05, 1.15, 1.19, 1.21, 1.28),
    (128, 448): (0.96, 1.03, 1.11, 1.15, 1.17, 1.20, 1.26),
    (128, 504): (1.01, 1.09, 1.15, 1.16, 1.17, 1.19, 1.24),
    (128, 672): (1.16, 1.16, 1.11, 1.09, 1.12, 1.21, 1.23),
    (64, 256): (0.76, 0.76, 0.76, 0.75, 0.75, 0.81, 0.87),
    (64, 320): (0.77, 0.76, 0.76, 0.78, 0.82, 0.87, 0.87),
    (64, 352): (0.76, 0.77, 0.77, 0.80, 0.87, 0.89, 0.90),
    (64, 384): (0.79, 0.78, 0.80, 0.85, 0.92, 0.92, 0.93),
    (64, 392): (0.78, 0.80, 0.86, 0.91, 0.97, 1.03, None),
    (64, 416): (0.79, 0.81, 0.86, 0.92, 0.99, 1.04, 1.09),
    (64, 448): (0.82, 0.84, 0.89, 0.96, 1.01, 1.05, 1.09),
    (64, 480): (0.82, 0.86, 0.93, 1.00, 1.02, 1.06, 1.09),
    (64, 490): (0.86, 0.90, 0.98, 1.02, 1.05, None, None),
    (64, 504): (0.87, 0.92, 0.98, 1.02, 1.05, None, None),
    (64, 512): (0.93, 1.01, 1.09, 1.12, 1.14, 1.19, 1.23),
    (64, 544): (0.96, 1.03, 1.09, 1.09, 1.07, 1.05, 1.04),
    (64, 546): (0.98, 1.06, 1.11, 1.13, 1.10, None, None),
}


def test_rule_follows_the_measurements(tmp_path):
    calls = [(d, jobs, s, r) for (d, jobs), rs in MEASURED.items() for s, r in zip(SHARES, rs) if r]
    body = "\n".join(f'putchar(daf::narrow_pays({d}, {jobs}, {s}) ? \'1\' : \'0\');' for d, jobs, s, _ in calls)
    src = tmp_path / "rule.cpp"
    src.write_text(f'#include <cstdio>\n#include "block_rule.h"\nint main() {{\n{body}\n}}\n')
    exe = tmp_path / "rule"
    inc = os.path.join(ROOT, "paper_2607_21599_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", f"-I{inc}", str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    for (d, jobs, s, r), c in zip(calls, got):
        if abs(r - 1.0) > 0.025:  # either height is right where they are level
            assert (c == "1") == (r < 1.0), (d, jobs, s, r)
