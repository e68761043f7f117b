"""GPU: the value range and the LSE of the bf16 attention kernels, against the
oracle. Probabilities are 1 at a row's reference score, so the fp32 sums
represent values of any normal magnitude; include/daf.h states the upper bound."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import daf_inputs as di
from parity import assert_attn_close, oracle_request

pytestmark = pytest.mark.gpu


def _layer(shape, arrays):
    """Both stages by their own calls; the outputs as float64."""
    from paper_2607_21599_amd.tensors import LayerBuffers
    batch = di.make_batch([shape])
    arrays(batch.arrays)
    buf = LayerBuffers(batch.arrays, batch.cu_doc, batch.cu_q, batch.cu_imp, shape.hq, shape.hkv, shape.d)
    buf.fuse_kv()
    buf.stage1()
    buf.stage2()
    torch.cuda.synchronize()
    out = {k: buf[k].float().cpu().numpy().astype(np.float64) for k in ("o_imp", "lse_imp", "o_q", "lse_q")}
    return out, batch.request(0)


@pytest.mark.parametrize("log2_scale,jump", [(-118, 20), (-100, 20), (84, 46)])
@pytest.mark.parametrize("n,d,back", [(150, 128, 20), (300, 64, 33), (2200, 128, 33), (2200, 128, 20)])
def test_values_of_any_magnitude(n, d, back, log2_scale, jump):
    """Values of 2^-118 (outputs of 2^-124 are still normal) to 2^84, with a key
    `jump` log2 units above the rest late in the sequence (64-row and 128-row
    blocks; an even and an odd key): the outputs are as close as those of values
    of order one. 2^46 times values of 2^84 would overflow: that key raises the
    reference."""
    def scale(a):
        for k, rows in (("v_imp", n), ("v_q", 40), ("v_cache", n + 900)):
            a[k][:rows] = di.f32_to_bf16_bits(di.raw_to_f32(a[k][:rows]) * np.float32(2.0 ** log2_scale))
        u = np.full(d, 1.0 / np.sqrt(d), np.float32)
        a["q_imp"] = di.f32_to_bf16_bits(di.raw_to_f32(a["q_imp"]) + np.float32(8.0) * u)
        k = di.raw_to_f32(a["k_imp"])
        k[n - back] = np.float32(jump * np.log(2.0) / 8.0 * np.sqrt(d)) * u
        a["k_imp"] = di.f32_to_bf16_bits(k)
    got, req = _layer(di.Shape("range", L_d=n + 900, L_q=40, n=n, hq=28, hkv=4, d=d, seed=n + d), scale)
    rows = np.unique(np.r_[0:n:max(1, n // 40), n - 40:n])
    ref = oracle_request(req, rows1=rows)
    for name, g, r in (("stage 1", got["o_imp"][rows], ref["o_imp"]), ("stage 2", got["o_q"], ref["o_q"])):
        assert_attn_close(g * 2.0 ** -log2_scale, r * 2.0 ** -log2_scale, di.BF16, f"{name}, values 2^{log2_scale}")


@pytest.mark.parametrize("n,L_d,loud", [(64, 300, 40), (128, 300, 100), (2200, 2300, 2180), (64, 100, 0)])
def test_lse_of_a_dominating_key_in_a_masked_tile(n, L_d, loud):
    """One key 18.49 log2 units above all others (scores of 0), first met in a
    row's masked tile: in stage 1 at `loud`, in stage 2 (loud 0) question token
    10. 2^0.49 is not a bf16 number, so the key's probability is exact only
    against its own score. What is left are the others' roundings, 2^-9 of at
    most 2200 x 2^-18.49, and fp32's: the bar is 1e-4 (a rounding of the key's
    own probability is 1e-3)."""
    d = 128

    def arrays(a):
        q = np.zeros(d, np.float32)
        q[0] = 8.0
        for k in ("q_imp", "q_q"):
            a[k][:] = di.f32_to_bf16_bits(q)
        for k in ("k_imp", "k_q", "k_cache"):
            a[k][:] = 0
        key = np.zeros(d, np.float32)
        key[0] = 18.125
        (a["k_imp"] if loud else a["k_q"])[loud or 10] = di.f32_to_bf16_bits(key)
    got, req = _layer(di.Shape("lse", L_d=L_d, L_q=20, n=n, hq=28, hkv=4, d=d, seed=n + loud), arrays)
    rows = np.arange(loud, n) if loud else np.arange(1)
    ref = oracle_request(req, rows1=rows)
    g, r = (got["lse_imp"].T[rows], ref["lse_imp"]) if loud else (got["lse_q"].T[10:], ref["lse_q"][10:])
    err = np.abs(g - r).max()
    assert err <= 1e-4, err


def test_lse_error_of_short_splits():
    """Stage 2 of few key tiles, heads from a nearly uniform to a peaked softmax:
    the LSE's error against 64 bits (2-norm over 24 inputs) is not above the 1.03e-5
    that one 64-key tile per split shows here; a reference that is raised only past
    2^28 gives more with the longer splits."""
    import paper_2607_21599_amd as daf
    L_d, L_q, hq, hkv, d = 1473, 243, 8, 2, 64
    cfg, batch = daf.AttnCfg(hq, hkv, d, daf.DAF_BF16), daf.Batch.single(L_d, L_q, 0)
    ws_bytes = daf.daf_qdoc_workspace_size(cfg, batch)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    scale = (8.0 ** (torch.arange(hq, device="cuda") / (hq - 1)))[:, None]
    mask = torch.arange(L_d + L_q, device="cuda")[None, :] > L_d + torch.arange(L_q, device="cuda")[:, None]
    num = den = 0.0
    for seed in range(24):
        g = torch.Generator(device="cuda").manual_seed(seed)
        q, k, v = (torch.empty((n, h, d), device="cuda").normal_(0.0, 0.5, generator=g)
                   for n, h in ((L_q, hq), (L_d + L_q, hkv), (L_d + L_q, hkv)))
        q, k, v = (q * scale).bfloat16(), k.bfloat16(), v.bfloat16()
        o, lse = torch.zeros_like(q), torch.zeros((hq, L_q), device="cuda")
        daf.daf_qdoc_attn(cfg, batch, q, k, v, o, lse, ws, ws_bytes)
        for h in range(hq):
            s = torch.mm(q[:, h].double().contiguous(), k[:, h * hkv // hq].double().t().contiguous()) / d ** 0.5
            ref = torch.logsumexp(s.masked_fill_(mask, -float("inf")), 1)
            num += float(((lse[h].double() - ref) ** 2).sum())
            den += float((ref ** 2).sum())
    assert (num / den) ** 0.5 <= 1.03e-5, (num / den) ** 0.5
