"""GPU: the decoder layer where its projections run in pieces along k, summed
with bias and residual by a second kernel, against the oracle. test_gemm_plan.py
pins what each row count runs: last rows only (100), halves and last rows (300,
640), Q, K and V with bias in 8, 4, 3 and 2 pieces, whole tiles before pieces
(5134)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import daf_inputs as di
import test_gpu_layer as tl
from oracle import decoder as dec
from oracle import get as oracle_get

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L_d,L_q,n", [(700, 20, 80), (900, 30, 270), (1500, 64, 436), (1200, 100, 540)])
def test_few_rows(L_d, L_q, n):
    tl.test_decoder_layer_daf(di.QWEN7B, L_d, L_q, n)


def test_whole_tiles_then_pieces():
    """5134 rows, every row recomputed: the output and down projections run 256
    whole tiles, then the last 24 (rows 4096 to 5119, columns from 2048) as
    halves and the 14 last rows in 4 pieces along k. Sampled rows of both."""
    import paper_2607_21599_amd as daf
    model, L_d, L_q = di.QWEN7B, 5100, 34
    T = L_d + L_q
    x, _, _, _, wts = tl._layer_setup(model, L_d, L_q, 1, seed=21)
    cfg = daf.AttnCfg(model.hq, model.hkv, model.d, daf.DAF_BF16)
    batch = daf.Batch.single(L_d, L_q, 0)
    w = tl._weights_on_gpu(model, wts)
    xa, pos = tl._dev(x), tl._dev(np.arange(T, dtype=np.int32))
    ws_bytes = daf.daf_decoder_layer_workspace_size(cfg, w, batch, daf.DAF_LAYER_FULL)
    ws = torch.full((ws_bytes,), 0xff, dtype=torch.uint8, device="cuda")  # NaNs
    daf.daf_decoder_layer(cfg, w, batch, daf.DAF_LAYER_FULL, None, pos, xa, None, None, ws, ws_bytes)
    torch.cuda.synchronize()
    rng = np.random.Generator(np.random.PCG64(5))
    rows = np.unique(np.r_[0, 4095, 4096, 4223, 4224, 5119, 5120, T - 1, rng.choice(np.arange(4096, T), 16, replace=False),
                           rng.choice(4096, 8, replace=False)])
    f, ow = di.raw_to_f32, tl._oracle_weights(wts)
    xf = f(x)
    h = dec.rmsnorm(xf, ow["w_in"], model.eps)
    k = dec.rope(dec.linear(h, ow["wk"], ow["bk"]).reshape(T, model.hkv, model.d), np.arange(T), model.theta)
    v = dec.linear(h, ow["wv"], ow["bv"]).reshape(T, model.hkv, model.d)
    q = dec.rope(dec.linear(h[rows], ow["wq"], ow["bq"]).reshape(len(rows), model.hq, model.d), rows, model.theta)
    o = oracle_get().position_attention(q.astype(np.float32), k.astype(np.float32), v.astype(np.float32), rows,
                                        1.0 / np.sqrt(model.d))[0].reshape(len(rows), -1)
    x1 = dec.linear(o, ow["wo"], residual=xf[rows])
    h2 = dec.rmsnorm(x1, ow["w_post"], model.eps)
    ref = dec.linear(dec.silu_mul(dec.linear(h2, ow["wg"]), dec.linear(h2, ow["wu"])), ow["wd"], residual=x1)
    tl._layer_close(tl._f(xa[torch.from_numpy(rows).cuda()]), ref, "5134 rows")
