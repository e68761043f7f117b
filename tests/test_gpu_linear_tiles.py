"""GPU: the projections at the edges of their tiling, and the rotary embedding on
either side of its vector rule, against the CPU oracle.

Ragged last rows on either side of 128, column counts that end inside a
256-column tile, one, odd and even k step counts, and launches with whole tiles
before cut ones (more than 256 tiles of 256 rows). daf_linear runs all but its two
largest sizes here in 128 x 128 tiles; test_gpu_linear_small.py has such edges for
the 256-row kernel, and so has the gated product. Outputs are
bf16 of order-1 values: half a bf16 ulp (2^-9 relative) plus fp32 accumulation,
checked as |gpu - oracle| <= 2^-8 |oracle| + 2e-3."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import daf_inputs as di
from oracle import decoder as dec

pytestmark = pytest.mark.gpu


def _dev(raw):
    from paper_2607_21599_amd.tensors import to_device
    return to_device(raw)


def _check(got, ref, what):
    got = got.float().cpu().numpy().astype(np.float64)
    bad = np.abs(got - ref) > 2.0 ** -8 * np.abs(ref) + 2e-3
    assert not bad.any(), f"{what}: {bad.sum()} of {bad.size} beyond the bf16 bar, first at {np.argwhere(bad)[0]}"


@pytest.mark.parametrize("M,N,K,bias,res", [
    (1, 128, 64, True, True), (127, 384, 64, False, True), (128, 256, 128, True, False), (129, 256, 192, True, True),
    (255, 640, 64, False, False), (257, 128, 320, True, True), (385, 512, 192, False, True),
    (700, 2304, 128, True, False),
    # 272 tiles of 256 rows: 256 whole, 16 cut in two, then one row range of 104 or none
    (4200, 4352, 64, True, True), (4226, 4096, 192, False, True),
    (5134, 2048, 128, True, False)])
def test_linear_tiles(M, N, K, bias, res):
    import paper_2607_21599_amd as daf
    A, W, b, R = di.make_linear_case(M, N, K, seed=M + N + K, bias=bias, residual=res)
    w = di.raw_to_f32
    ref = dec.linear(w(A), w(W), None if b is None else w(b), None if R is None else w(R))
    C = torch.full((M + 3, N), 7.0, dtype=torch.bfloat16, device="cuda")
    if res:
        C[:M] = _dev(R)
    daf.daf_linear(M, N, K, _dev(A), _dev(W), None if b is None else _dev(b), C if res else None, C)
    torch.cuda.synchronize()
    _check(C[:M], ref, f"linear {M}x{N}x{K}")
    assert torch.all(C[M:] == 7.0), "rows past M were written"


@pytest.mark.parametrize("M,I,K", [(1, 64, 64), (128, 128, 192), (130, 192, 64), (300, 320, 128),
                                   (4200, 2176, 64), (5134, 1024, 192)])
def test_swiglu_tiles(M, I, K):
    import paper_2607_21599_amd as daf
    A, Wgu, _, _ = di.make_linear_case(M, 2 * I, K, seed=M + I, bias=False, residual=False)
    C = torch.full((M + 3, I), 5.0, dtype=torch.bfloat16, device="cuda")
    daf.daf_linear_swiglu(M, I, K, _dev(A), _dev(Wgu), C)
    torch.cuda.synchronize()
    w = di.raw_to_f32
    ref = dec.silu_mul(dec.linear(w(A), w(Wgu)[:I]), dec.linear(w(A), w(Wgu)[I:]))
    _check(C[:M], ref, f"swiglu {M}x{I}x{K}")
    assert torch.all(C[M:] == 5.0), "rows past M were written"


@pytest.mark.parametrize("rows,heads,d,stride,shift", [
    (257, 28, 128, 4608, 0), (1, 9, 16, 144, 0), (6, 9, 64, 640, 0), (9, 3, 256, 776, 0),  # 16-byte pieces
    (1, 1, 16, 16, 0), (5, 3, 64, 192, 0), (9, 2, 256, 520, 0), (33, 8, 64, 512, 0), (10, 5, 128, 640, 0),  # few heads, and above
    (7, 3, 64, 196, 0), (6, 2, 128, 256, 1), (3, 2, 24, 48, 0), (4, 1, 512, 512, 0)])     # stride, address, sizes
def test_rope_paths(rows, heads, d, stride, shift):
    """Both rope kernels on either side of the rule that picks them; the rest
    of each row (and what lies before and after) stays."""
    import paper_2607_21599_amd as daf
    rng = np.random.Generator(np.random.PCG64(rows + d))
    raw = di.f32_to_bf16_bits(rng.standard_normal(rows * stride + 16, dtype=np.float32))
    pos = np.sort(rng.choice(131072, rows, replace=False)).astype(np.int32)
    t = _dev(raw)
    daf.daf_rope(rows, heads, d, stride, t[shift:], _dev(pos), 1e6)
    torch.cuda.synchronize()
    got = t.view(torch.int16).cpu().numpy().view(np.uint16)
    x = raw[shift:shift + rows * stride].reshape(rows, stride)
    ref = dec.rope(di.raw_to_f32(x)[:, :heads * d].reshape(rows, heads, d), pos, 1e6).reshape(rows, heads * d)
    g = got[shift:shift + rows * stride].reshape(rows, stride)
    err = np.abs(di.raw_to_f32(g)[:, :heads * d].astype(np.float64) - ref)
    assert (err <= 2.0 ** -8 * np.abs(ref) + 2e-3).all(), err.max()
    assert np.array_equal(g[:, heads * d:], x[:, heads * d:]), "past the heads"
    assert np.array_equal(got[:shift], raw[:shift]) and np.array_equal(got[shift + rows * stride:], raw[shift + rows * stride:])
