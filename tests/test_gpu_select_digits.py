"""The top-n kernel of daf_select_important at the edges of its digit passes, its
slabs and its waves' ranges: the chosen indices against a stable sort of the
scores that the call itself returns, exactly."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 64  # fp32 keys of one head: a score is the magnitude of a token's one deviating feature


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    import paper_2607_21599_amd as daf
    daf.lib()
    yield
    torch.cuda.synchronize()


def _values(kind, L, rng):
    if kind == "spread":  # every digit width down to the last bits
        return np.exp(rng.uniform(-20, 5, L))
    if kind == "narrow":  # many keys share the digits of three passes
        return 1.0 + rng.integers(0, 2000, L) * 2.0**-23
    if kind == "zeros":  # ties at zero, which lanes past the last token hold too
        return np.where(rng.random(L) < 0.3, rng.random(L), 0.0)
    if kind == "few":  # large groups of equal keys across waves and slabs
        return rng.integers(1, 6, L).astype(np.float64)
    return np.full(L, 2.5)  # "equal"


@pytest.mark.parametrize("kind", ["spread", "narrow", "zeros", "few", "equal"])
def test_topn_edges(kind):
    import paper_2607_21599_amd as daf
    rng = np.random.Generator(np.random.PCG64(len(kind)))
    lens = [1, 63, 64, 65, 511, 512, 513, 2047, 2048, 2049, 4100, 32767, 32768, 32769, 33000, 49153]
    for group in (lens[:13], lens[13:], lens):  # one slab, across slabs, both in one batch
        L = np.array(group)
        for frac in (0.0, 0.15, 0.5, 0.999, 1.0):
            n = np.maximum(1, np.minimum(L, np.round(frac * L).astype(int)))
            cu_doc, cu_imp = np.r_[0, np.cumsum(L)], np.r_[0, np.cumsum(n)]
            v = np.concatenate([_values(kind, int(x), rng) for x in L]).astype(np.float32)
            fresh = torch.zeros(len(v), 1, D)
            fresh[:, 0, 5] = torch.from_numpy(v)
            fresh, cached = fresh.cuda(), torch.zeros(len(v), 1, D, device="cuda")
            scores = torch.full((len(v),), -1.0, device="cuda")
            idx = torch.full((int(cu_imp[-1]),), -7, dtype=torch.int32, device="cuda")
            daf.daf_select_important(daf.AttnCfg(1, 1, D, daf.DAF_F32), daf.Batch(cu_doc, 0 * cu_doc, cu_imp),
                                     [fresh], [cached], scores, idx)
            torch.cuda.synchronize()
            s, got = scores.cpu().numpy(), idx.cpu().numpy()
            for b in range(len(L)):
                sb = s[cu_doc[b]:cu_doc[b + 1]]
                want = np.sort(np.argsort(-sb, kind="stable")[:n[b]])
                assert np.array_equal(got[cu_imp[b]:cu_imp[b + 1]], want), (kind, int(L[b]), int(n[b]))


@pytest.mark.parametrize("kind", ["spread", "few"])
def test_topn_slabs(kind):
    """Requests of two to seven slabs of equal size, alone and together."""
    import paper_2607_21599_amd as daf
    rng = np.random.Generator(np.random.PCG64(7))
    for L in ([32770], [65536], [65537], [98305], [131071], [200001], [70000, 300, 100000]):
        L = np.array(L)
        n = np.maximum(1, (L * 0.15).astype(int))
        cu_doc, cu_imp = np.r_[0, np.cumsum(L)], np.r_[0, np.cumsum(n)]
        fresh = torch.zeros(int(cu_doc[-1]), 1, D)
        fresh[:, 0, 5] = torch.from_numpy(_values(kind, int(cu_doc[-1]), rng).astype(np.float32))
        fresh, cached = fresh.cuda(), torch.zeros(int(cu_doc[-1]), 1, D, device="cuda")
        scores = torch.full((int(cu_doc[-1]),), -1.0, device="cuda")
        idx = torch.full((int(cu_imp[-1]),), -7, dtype=torch.int32, device="cuda")
        daf.daf_select_important(daf.AttnCfg(1, 1, D, daf.DAF_F32), daf.Batch(cu_doc, 0 * cu_doc, cu_imp),
                                 [fresh], [cached], scores, idx)
        torch.cuda.synchronize()
        s, got = scores.cpu().numpy(), idx.cpu().numpy()
        for b in range(len(L)):
            want = np.sort(np.argsort(-s[cu_doc[b]:cu_doc[b + 1]], kind="stable")[:n[b]])
            assert np.array_equal(got[cu_imp[b]:cu_imp[b + 1]], want), (kind, int(L[b]))
