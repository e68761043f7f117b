"""CPU: inline assembly that writes the m0 register says so to the compiler, which
otherwise may keep a value of its own there across the block."""
from __future__ import annotations

import glob
import os
import re

from conftest import ROOT


def test_m0_is_a_declared_clobber():
    writers = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2607_21599_amd", "csrc", "*.h*"))):
        with open(path) as f:
            src = f.read()
        for block in re.findall(r"\basm\b[^(;]*\((.*?)\);", src, re.S):
            if re.search(r"\bs_\w+ m0,", block):
                writers += 1
                assert re.search(r'"m0"', block.rsplit(":", 1)[1]), f"{os.path.basename(path)}: {block.strip()[:60]}"
    assert writers, "no block that writes m0 was found"
