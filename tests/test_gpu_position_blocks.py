"""GPU: position attention around the block-height rule (64 or 128 rows, chosen
on the host or, for given positions, by the kernel), against the oracle: rows
spread over the keys, rows at their end (given and as NULL), job counts below,
inside and above the range where the positions decide."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import daf_inputs as di
import oracle as orc_mod
from parity import assert_attn_close, assert_lse_close, sample_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["spread", "end", "null"])
@pytest.mark.parametrize("rows,keys,hq,hkv,d", [
    (1100, 4000, 28, 4, 128), (1281, 5000, 28, 4, 128), (1700, 1900, 28, 4, 128), (2048, 9000, 28, 4, 128),
    (2049, 2600, 28, 4, 128),                           # 252, 308, 392, 448 and 476 jobs
    (6200, 7000, 8, 2, 64), (7168, 20000, 8, 2, 64), (8064, 9000, 8, 2, 64),  # 392, 448, 504
    (8192, 8400, 8, 2, 64), (8704, 8900, 8, 2, 64), (8705, 9000, 8, 2, 64),   # 512, 544, 552
    (2200, 3000, 18, 3, 128)])                          # 324, a KV head count that does not divide the 8 XCDs
def test_position_block_heights(rows, keys, hq, hkv, d, where):
    import paper_2607_21599_amd as daf
    from paper_2607_21599_amd.tensors import to_device
    rng = np.random.Generator(np.random.PCG64(rows + keys))
    pos = np.arange(keys - rows, keys)
    if where == "spread":
        pos = np.sort(rng.choice(keys, size=rows, replace=False))
    q, k, v = (di._normal(rng, (n, h, d), 0.5, di.BF16) for n, h in ((rows, hq), (keys, hkv), (keys, hkv)))
    tq, tk, tv = to_device(q), to_device(k), to_device(v)
    tp = None if where == "null" else to_device(pos.astype(np.int32))
    o = torch.full((rows + 1, hq, d), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((hq, rows), dtype=torch.float32, device="cuda")
    daf.daf_position_attn(daf.AttnCfg(hq, hkv, d, daf.DAF_BF16), rows, keys, tq, tp, tk, tv, o, lse)
    torch.cuda.synchronize()
    at = sample_rows(rows, 32, seed=rows, tile=64)
    w = di.raw_to_f32
    ro, rl = orc_mod.get().position_attention(w(q)[at], w(k), w(v), pos[at], orc_mod.default_scale(d))
    assert_attn_close(o[:rows].float().cpu().numpy()[at], ro, di.BF16, where)
    assert_lse_close(lse.cpu().numpy().T[at], rl, di.BF16, where)
    assert torch.all(o[rows] == 7.0), "past the last row"
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    assert (o[:rows].float().abs().amax(dim=(1, 2)) > 0).all(), "a row was not written"
