"""GPU: stage 1 on either side of the block-height rule, against the oracle.

Launches of up to 448 (128-row block, head) pairs (D = 64: 544; see
test_gpu_position_blocks.py) run 64-row blocks, larger ones 128-row blocks: row
counts just below and above the line for several head shapes, sizes that end
inside a block, a ragged batch, and queries and keys that make the running
reference rise late (each loud key 40 log2 units above the one before). The bars are those of tests/parity.py."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import daf_inputs as di
from parity import assert_attn_close, assert_lse_close, oracle_request, sample_rows

pytestmark = pytest.mark.gpu


def _run(shapes, loud=()):
    from paper_2607_21599_amd.tensors import LayerBuffers
    batch = di.make_batch(shapes)
    s0 = shapes[0]
    if loud:
        u = np.full(s0.d, 1.0 / np.sqrt(s0.d), np.float32)
        a = batch.arrays
        a["q_imp"] = di.f32_to_bf16_bits(di.raw_to_f32(a["q_imp"]) + np.float32(8.0) * u)
        k = di.raw_to_f32(a["k_imp"])
        for j, pos in enumerate(loud):
            k[pos] = np.float32(40.0 * (j + 1) * np.sqrt(s0.d / 128.0)) * u
        a["k_imp"] = di.f32_to_bf16_bits(k)
    buf = LayerBuffers(batch.arrays, batch.cu_doc, batch.cu_q, batch.cu_imp, s0.hq, s0.hkv, s0.d)
    buf.stage1()
    torch.cuda.synchronize()
    o, lse = buf["o_imp"].float().cpu().numpy(), buf["lse_imp"].cpu().numpy().T
    for b, s in enumerate(shapes):
        rows = sample_rows(s.n, 48, seed=s.n, tile=64)
        ref = oracle_request(batch.request(b), rows1=rows, want=("s1",))
        at = int(batch.cu_imp[b]) + rows
        assert_attn_close(o[at], ref["o_imp"], di.BF16, f"n={s.n} request {b}")
        assert_lse_close(lse[at], ref["lse_imp"], di.BF16, f"n={s.n} request {b} lse")


@pytest.mark.parametrize("n,hq,hkv,d", [
    (2048, 28, 4, 128), (2049, 28, 4, 128),  # 448 and 476 blocks
    (4096, 14, 2, 128), (4097, 14, 2, 128), (7168, 8, 2, 64), (7169, 8, 2, 64),
    (15, 28, 4, 128), (65, 6, 3, 64), (193, 5, 5, 128)])
def test_stage1_block_height(n, hq, hkv, d):
    _run([di.Shape(f"blk{n}", L_d=n + 7, L_q=1, n=n, hq=hq, hkv=hkv, d=d, seed=300 + n)])


def test_stage1_block_height_ragged():
    ns = (333, 64, 500, 1, 129)  # 10 blocks of 128 rows and 28 heads: 64-row blocks
    _run([di.Shape(f"r{i}", L_d=n + 3, L_q=1, n=n, seed=50 + i) for i, n in enumerate(ns)])


@pytest.mark.parametrize("n", [700, 2200])
def test_stage1_reference_raised_late(n):
    _run([di.Shape("loud", L_d=n + 5, L_q=1, n=n, seed=9)], loud=(70, n // 3, n // 2 + 1))


@pytest.mark.parametrize("reqs,hq,hkv,d,dtype", [
    ([(4000, 128, 300)], 28, 4, 128, di.BF16),   # one launch, stage 2 first (its jobs are the longer ones)
    ([(3000, 8, 900)], 28, 4, 128, di.BF16),     # one launch, stage 1 first
    ([(2500, 40, 1200), (300, 9, 5), (64, 70, 0), (700, 0, 100)], 8, 2, 64, di.BF16),
    ([(900, 33, 200), (500, 5, 130)], 4, 1, 64, di.F32),
    ([(700, 20, 90)], 14, 2, 128, di.F32),
    ([(200 + 10 * i, 3 + i, 20 + i) for i in range(20)], 7, 1, 128, di.BF16),  # 40 entries: two launches
    ([(2100, 16, 2048)], 28, 4, 128, di.BF16), ([(2100, 16, 2049)], 28, 4, 128, di.BF16),  # the rule's line
    ([(9000, 130, 2300)], 28, 4, 128, di.BF16), ([(30000, 97, 2300), (700, 3, 65)], 28, 4, 128, di.BF16)])
def test_layer_equals_stage_calls(reqs, hq, hkv, d, dtype):
    """The layer call in each launch form writes what the stage calls write,
    bit for bit, and the stage calls' outputs are the oracle's."""
    from paper_2607_21599_amd.tensors import LayerBuffers
    shapes = [di.Shape(f"l{i}", L_d=r[0], L_q=r[1], n=r[2], hq=hq, hkv=hkv, d=d, dtype=dtype, seed=700 + i)
              for i, r in enumerate(reqs)]
    batch = di.make_batch(shapes)
    a, b = (LayerBuffers(batch.arrays, batch.cu_doc, batch.cu_q, batch.cu_imp, hq, hkv, d) for _ in range(2))
    a["ws"].fill_(0xff)  # the workspace starts as NaNs
    a.layer()
    b.fuse_kv()
    b.stage1()
    b.stage2()
    b.fuse_hidden()
    torch.cuda.synchronize()
    for k in ("o_imp", "o_q", "lse_imp", "lse_q", "hidden", "k_cache", "v_cache"):
        assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k
    for i, s in enumerate(shapes[:4]):
        rows = sample_rows(s.n, 24, seed=s.n)
        ref = oracle_request(batch.request(i), rows1=rows)
        if s.n:
            assert_attn_close(b["o_imp"].float().cpu().numpy()[int(batch.cu_imp[i]) + rows], ref["o_imp"], dtype, "stage 1")
        if s.L_q:
            q = slice(int(batch.cu_q[i]), int(batch.cu_q[i + 1]))
            assert_attn_close(b["o_q"].float().cpu().numpy()[q], ref["o_q"], dtype, "stage 2")
