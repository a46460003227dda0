"""Attention (Fig. 1, right) where the kernels change their work split,
against the fp64 oracle: grids of few query blocks, whose workgroups split
the keys between waves, with empty, short, odd, long (past one register of
list entries) and full lists; and the sizes on both sides of the split."""
import numpy as np
import pytest

import oracle
import workloads as W

from .helpers import OUT_MAX_ABS, OUT_MEAN_ABS, dev_bf16, host_f32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2503_16428_amd as X  # noqa: E402


def _lists(hq, NB, causal, rng):
    """Row r holds 0, 1, 2, 3, 4, 5, 64, 65 .. or all of its candidates."""
    lengths = [0, 1, 2, 3, 4, 5, 63, 64, 65, 66, NB]
    idx = np.full((hq * NB, NB), -1, np.int32)
    cnt = np.zeros(hq * NB, np.int32)
    for r in range(hq * NB):
        cand = r % NB + 1 if causal else NB
        n = min(cand, lengths[(r + r // NB) % len(lengths)])
        sel = np.sort(rng.choice(cand, n, replace=False))
        idx[r, :n] = sel
        cnt[r] = n
    return idx, cnt


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("hq,hkv,NB", [(1, 1, 1), (1, 1, 2), (3, 1, 5), (2, 2, 32), (4, 2, 16),
                                       (5, 1, 13), (1, 1, 100), (2, 1, 64), (3, 3, 43)])
def test_lists_of_every_length(hq, hkv, NB, causal):
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=hq, hkv=hkv, seed=600 + NB))
    idx, cnt = _lists(hq, NB, causal, np.random.default_rng(NB))
    q, k, v = (dev_bf16(x[n]) for n in "qkv")
    di = torch.from_numpy(idx.reshape(hq, NB, NB)).cuda()
    dc = torch.from_numpy(cnt.reshape(hq, NB)).cuda()
    print(f"attn edge hq={hq} hkv={hkv} NB={NB} causal={causal}", flush=True)
    o, lse = X.xattn_block_sparse_attn(q, k, v, di, dc, causal=causal)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.sparse_attn_rows(x["q"], x["k"], x["v"], 128, idx, cnt, causal)
    og, lg = host_f32(o).reshape(o_ref.shape), host_f32(lse).reshape(lse_ref.shape)
    empty = ~np.isfinite(lse_ref)
    assert np.all(og[empty] == 0) and np.all(np.isneginf(lg[empty]))
    if not empty.all():
        e = np.abs(og.astype(np.float64) - o_ref)[~empty]
        print(f"  max_abs={e.max():.3e} mean_abs={e.mean():.3e}", flush=True)
        assert e.max() <= OUT_MAX_ABS and e.mean() <= OUT_MEAN_ABS
    np.testing.assert_allclose(lg[~empty], lse_ref[~empty], rtol=2e-3, atol=2e-2)

    full = np.tile(np.arange(NB, dtype=np.int32), (hq, NB, 1))
    n = np.tile(np.arange(1, NB + 1) if causal else np.full(NB, NB), (hq, 1)).astype(np.int32)
    o1, l1 = X.xattn_block_sparse_attn(q, k, v, torch.from_numpy(full).cuda(),
                                       torch.from_numpy(n).cuda(), causal=causal)
    o2, l2 = X.xattn_dense_attn(q, k, v, causal=causal)
    o3, l3 = X.xattn_dense_attn(q, k, v, causal=causal)
    torch.cuda.synchronize()
    for a, b in ((o1, o2), (o2, o3)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert torch.equal(l1, l2) and torch.equal(l2, l3)
    o_ref, _ = oracle.dense_attn_rows(x["q"], x["k"], x["v"], 128, causal)
    e = np.abs(host_f32(o2).reshape(o_ref.shape).astype(np.float64) - o_ref)
    assert e.max() <= OUT_MAX_ABS and e.mean() <= OUT_MEAN_ABS


@pytest.mark.parametrize("hq,NB", [(1, 7), (16, 9)])
def test_malformed_lists_stay_in_bounds(hq, NB):
    """Entries and counts out of range are clamped, as before: finite outputs, no fault."""
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=hq, hkv=1, seed=640))
    q, k, v = (dev_bf16(x[n]) for n in "qkv")
    idx = torch.full((hq, NB, NB), 10 ** 6, dtype=torch.int32, device="cuda")
    idx[:, :, ::2] = -5
    cnt = torch.full((hq, NB), NB + 9, dtype=torch.int32, device="cuda")
    cnt[:, 0] = -3
    o, _ = X.xattn_block_sparse_attn(q, k, v, idx, cnt, causal=False)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and (o[:, :128] == 0).all()


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("hq,NB", [(1, 1), (2, 5), (1, 50)])
def test_products_that_overflow(hq, NB, causal):
    """A query whose products with one wave's first keys are -inf gives them no weight."""
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=hq, hkv=1, seed=660))
    big = int(np.float32(3e38).view(np.uint32) >> 16)
    q, k = x["q"].copy(), x["k"].copy()
    q[..., 0] = 0
    k[..., 0] = 0
    q[..., 40::61, 0] = big
    k[..., :32, 0] = big | 0x8000
    print(f"attn overflow hq={hq} NB={NB} causal={causal}", flush=True)
    o, lse = X.xattn_dense_attn(dev_bf16(q), dev_bf16(k), dev_bf16(x["v"]), causal=causal)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.dense_attn_rows(q, k, x["v"], 128, causal)
    e = np.abs(host_f32(o).reshape(o_ref.shape).astype(np.float64) - o_ref)
    assert e.max() <= OUT_MAX_ABS and e.mean() <= OUT_MEAN_ABS
    np.testing.assert_allclose(host_f32(lse).reshape(lse_ref.shape), lse_ref, rtol=2e-3, atol=2e-2)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("hq,hkv,NB", [(1, 1, 1), (1, 1, 2), (1, 1, 7), (2, 1, 5), (1, 1, 50),
                                       (16, 2, 9), (3, 1, 50)])
def test_infinite_values_reach_their_queries_alone(hq, hkv, NB, causal):
    """A value of +-inf at a visible key gives +-inf in its feature and nothing in the others,
    on both sides of the split (the last two grids are past it) and for lists of every length."""
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=hq, hkv=hkv, seed=680 + NB))
    # inputs a tenth as large: every visible key keeps a weight above 0
    q, k = (W.to_bf16_bits(0.1 * W.bf16_bits_to_f32(x[n])) for n in "qk")
    v, zero = x["v"].copy(), x["v"].copy()
    inf = int(np.float32(np.inf).view(np.uint32) >> 16)
    v[:, ::128, 5], v[:, ::128, 77] = inf, inf | 0x8000  # the first key of a block: all see it
    zero[:, ::128, 5] = zero[:, ::128, 77] = 0
    idx, cnt = _lists(hq, NB, causal, np.random.default_rng(NB))
    full = np.tile(np.arange(NB, dtype=np.int32), (hq * NB, 1))
    n = np.tile(np.arange(1, NB + 1) if causal else np.full(NB, NB), hq).astype(np.int32)
    rest = np.setdiff1d(np.arange(128), [5, 77])
    for tag, ix, ct in (("lists", idx, cnt), ("full", full, n)):
        print(f"attn inf hq={hq} NB={NB} causal={causal} {tag}", flush=True)
        o, _ = X.xattn_block_sparse_attn(
            dev_bf16(q), dev_bf16(k), dev_bf16(v), torch.from_numpy(ix.reshape(hq, NB, NB)).cuda(),
            torch.from_numpy(ct.reshape(hq, NB)).cuda(), causal=causal)
        torch.cuda.synchronize()
        o_ref, _ = oracle.sparse_attn_rows(q, k, zero, 128, ix, ct, causal)
        og = host_f32(o).reshape(o_ref.shape)
        some = ct > 0
        assert np.all(np.isposinf(og[some][..., 5])) and np.all(np.isneginf(og[some][..., 77]))
        e = np.abs(og[..., rest].astype(np.float64) - o_ref[..., rest])
        assert e.max() <= OUT_MAX_ABS and e.mean() <= OUT_MEAN_ABS


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("spoiled", [64, 128, 200])
@pytest.mark.parametrize("hq,NB", [(2, 5), (1, 50), (16, 9), (3, 50)])
def test_products_that_overflow_over_whole_tiles(hq, NB, spoiled, causal):
    """As above with every key of the first half-tile, block or more: a query has seen only
    -inf when another query of its wave moves its reference. The last two grids run
    128-query workgroups."""
    L = 128 * NB
    x = W.generate(W.small("edge", L, hq=hq, hkv=1, seed=670))
    big = int(np.float32(3e38).view(np.uint32) >> 16)
    q, k = x["q"].copy(), x["k"].copy()
    q[..., 0] = 0
    k[..., 0] = 0
    q[..., 261::61, 0] = big  # queries that see keys past the spoiled ones
    k[..., :spoiled, 0] = big | 0x8000
    print(f"attn overflow hq={hq} NB={NB} spoiled={spoiled} causal={causal}", flush=True)
    o, lse = X.xattn_dense_attn(dev_bf16(q), dev_bf16(k), dev_bf16(x["v"]), causal=causal)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.dense_attn_rows(q, k, x["v"], 128, causal)
    e = np.abs(host_f32(o).reshape(o_ref.shape).astype(np.float64) - o_ref)
    assert e.max() <= OUT_MAX_ABS and e.mean() <= OUT_MEAN_ABS
    np.testing.assert_allclose(host_f32(lse).reshape(lse_ref.shape), lse_ref, rtol=2e-3, atol=2e-2)
