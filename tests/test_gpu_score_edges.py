"""Block scores (Algorithm 1) where the kernels change their work split,
against the fp64 oracle on sampled rows: rows whose sub-tile factors fit one
LDS stage of the finalisation exactly, exceed it by one sub-tile, and take
several stages; every kernel of the partial sums (stride, causal or not, tile
size) at a ragged length."""
import numpy as np
import pytest

import oracle
import workloads as W

from .helpers import compare_scores, dev_bf16, host_f32
from .score_tiles import CASES, CUS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2503_16428_amd as X  # noqa: E402


def _check(NB, hq, S, causal, seed, batch=1):
    """Two heads of queries, repeated to hq heads on one key head."""
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=2, hkv=1, seed=seed))
    q, k = dev_bf16(x["q"]), dev_bf16(x["k"])
    n = max(1, hq // 2)
    q, k = q[:hq].repeat(batch * n, 1, 1)[:batch * hq], k.repeat(batch, 1, 1)
    if batch > 1:
        q, k = q.view(batch, hq, L, 128), k.view(batch, 1, L, 128)
    print(f"score edge NB={NB} hq={hq} S={S} causal={causal} batch={batch}", flush=True)
    sc = X.xattn_score(q, k, causal=causal, stride=S)
    torch.cuda.synchronize()
    heads = min(hq, 2)
    for h in range(hq * batch):  # equal inputs, whatever tile or compute unit they ran on
        assert torch.equal(sc[h], sc[h % heads]), h
    b = np.unique(np.clip([0, 1, NB // 3, NB // 2, NB - 2, NB - 1], 0, NB - 1))
    rh = np.repeat(np.arange(heads), len(b)).astype(np.int32)
    rb = np.tile(b, heads).astype(np.int32)
    want = oracle.score_rows(x["q"], x["k"], 128, S, causal, rows=(rh, rb))
    got = host_f32(sc[:heads])[rh, rb]
    rep = compare_scores(got, want)
    print(f"  {rep}", flush=True)
    assert rep["n_bad"] == 0
    np.testing.assert_allclose(got.sum(-1), 1.0, atol=1e-4)
    if causal:
        assert np.all(got[np.arange(NB)[None, :] > rb[:, None]] == 0)


# S = 1: 128 reduced rows, 32 sub-tiles a stage; S = 2: 64 rows, 64 sub-tiles
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,NB", [(1, 32), (1, 33), (1, 65), (2, 128), (2, 129)])
def test_rows_longer_than_one_factor_stage(S, NB, causal):
    _check(NB, 1, S, causal, seed=900 + NB + S)


# reduced lengths below, at and just past 32, 64, 128 and 256 rows at every stride, from one
# head to many (each kernel by its name: test_every_kernel)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S", [1, 2, 4, 8, 16, 32, 64])
def test_every_tile_size(S, causal):
    for hq, NB in [(1, 1), (1, 2), (2, 3), (1, 17), (8, 5), (16, 9), (32, 9), (32, 33), (32, 65)]:
        if NB * hq * (8 // min(S, 8)) <= 32 * 65 * 2:
            _check(NB, hq, S, causal, seed=950 + NB)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,NB,hq", [(2, 65, 8), (4, 129, 8), (16, 257, 16), (32, 300, 32),
                                     (64, 600, 32)])
def test_ragged_256_row_tiles(S, NB, hq, causal):
    _check(NB, hq, S, causal, seed=980 + NB)


def test_batches_on_small_tiles():
    _check(37, 8, 16, True, seed=990, batch=3)


@pytest.mark.parametrize("S,causal,tile,hq,NB", CASES)
def test_every_kernel(S, causal, tile, hq, NB):
    if torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8 != CUS:
        pytest.skip(f"the shapes are for {CUS} compute units")
    _check(NB, hq, S, causal, seed=1000 + NB)
