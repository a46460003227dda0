"""Block scores (Algorithm 1) where the kernels change their work split,
against the fp64 oracle on sampled rows: rows whose sub-tile factors fit one
LDS stage of the finalisation exactly, exceed it by one sub-tile, and take
several stages."""
import numpy as np
import pytest

import oracle
import workloads as W

from .helpers import compare_scores, dev_bf16, host_f32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2503_16428_amd as X  # noqa: E402


def _check(NB, hq, hkv, S, causal, seed, batch=1):
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=hq * batch, hkv=hkv * batch, seed=seed))
    q, k = dev_bf16(x["q"]), dev_bf16(x["k"])
    if batch > 1:
        q, k = q.view(batch, hq, L, 128), k.view(batch, hkv, L, 128)
    print(f"score edge NB={NB} hq={hq} hkv={hkv} S={S} causal={causal} batch={batch}", flush=True)
    sc = X.xattn_score(q, k, causal=causal, stride=S)
    torch.cuda.synchronize()
    b = np.unique(np.clip([0, 1, NB // 2, NB - 2, NB - 1], 0, NB - 1))
    heads = np.arange(hq * batch)
    rh = np.repeat(heads, len(b)).astype(np.int32)
    rb = np.tile(b, len(heads)).astype(np.int32)
    want = oracle.score_rows(x["q"], x["k"], 128, S, causal, rows=(rh, rb))
    got = host_f32(sc)[rh, rb]
    rep = compare_scores(got, want)
    print(f"  {rep}", flush=True)
    assert rep["n_bad"] == 0
    np.testing.assert_allclose(host_f32(sc).sum(-1), 1.0, atol=1e-4)
    if causal:
        assert np.all(got[np.arange(NB)[None, :] > rb[:, None]] == 0)


# S = 1: 128 reduced rows, 32 sub-tiles a stage; S = 2: 64 rows, 64 sub-tiles
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,NB", [(1, 32), (1, 33), (1, 65), (2, 128), (2, 129)])
def test_rows_longer_than_one_factor_stage(S, NB, causal):
    _check(NB, 1, 1, S, causal, seed=900 + NB + S)
