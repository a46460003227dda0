"""Block selection (find_blocks, Top-K, Top-Ratio) bit for bit against the
oracle on rows that stress the search: one repeated mass, a few distinct
masses many times over, masses over the whole 32-bit range, scores of exactly
1 and above, the values next to 1 and to 2^-32, zeros, negatives and NaN, at
row lengths around the slots of a wave."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2503_16428_amd as X  # noqa: E402


def _row(kind, n, rng):
    if kind == 0:
        return np.full(n, 1.0 / n)
    if kind == 1:
        return rng.choice([0.0, 2.0 ** -32, 2.0 ** -10, 3 * 2.0 ** -10, 0.25], n)
    if kind == 2:
        return 2.0 ** rng.uniform(-34, 0, n)
    if kind == 3:  # one block holds everything
        x = np.zeros(n)
        x[rng.integers(n)] = 1.0
        return x
    if kind == 4:
        return rng.choice([1.0, 1.5, 1.0 - 2.0 ** -24, 0.0, 0.5, 2.0 ** -33], n)
    if kind == 5:
        return rng.choice([np.nan, -1.0, 0.0, 0.125, 0.125 + 2.0 ** -26, 1e-7], n)
    if kind == 6:
        return np.zeros(n)
    if kind == 7:  # two tight clusters of neighbouring floats
        return np.where(rng.random(n) < 0.5, 0.5, 1e-3) * (1 + rng.integers(0, 3, n) * 2.0 ** -23)
    if kind == 8:
        return np.full(n, 1.0)
    return rng.dirichlet(np.full(n, 0.3))


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("NB", [1, 2, 63, 64, 65, 127, 129, 200, 257, 513, 1025, 1100])
def test_hard_rows(NB, causal):
    rng = np.random.default_rng(NB)
    H = 2
    full = np.zeros((H, NB, NB), np.float32)
    for h in range(H):
        for b in range(NB):
            full[h, b] = _row((b + 3 * h) % 10, NB, rng)
            if causal:  # what is not a candidate must not matter
                full[h, b, b + 1:] = 7.0
    sc = torch.from_numpy(full).cuda()
    dims = X.Dims(1, H, 1, NB * 128, 128, int(causal))
    clean = np.nan_to_num(full.astype(np.float64), nan=0.0).reshape(H * NB, NB)
    rb = np.tile(np.arange(NB, dtype=np.int32), H)
    print(f"select edge NB={NB} causal={causal}", flush=True)

    def check(got, want, what):
        gi, gc = (t.cpu().numpy() for t in got)
        oi, oc = want
        assert np.array_equal(gc.reshape(-1), oc), what
        assert np.array_equal(gi.reshape(H * NB, NB), oi), what

    for tau in (1e-6, 0.3, 0.9, 0.999999):
        check(X.xattn_select(sc, dims, tau), oracle.select_rows(clean, rb, tau, causal), tau)
    for k in (1, 2, 63, 64, 65, max(1, NB // 2), max(1, NB - 1)):
        check(X.xattn_select_topk(sc, dims, k), oracle.select_topk_rows(clean, rb, k, causal), k)
    check(X.xattn_select_ratio(sc, dims, 0.37),
          oracle.select_ratio_rows(clean, rb, 0.37, causal), "ratio")


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("hq,NB,tau", [(1, 1, 0.9), (1, 64, 0.9), (2, 65, 0.5), (3, 129, 0.95),
                                       (8, 256, 0.9), (16, 128, 0.9), (17, 128, 0.9), (1, 257, 0.9),
                                       (2, 33, 1.0)])
def test_forward_lists_are_the_selection_of_its_scores(hq, NB, tau, causal):
    """Rows few enough to be selected where they are finalised, and one past that."""
    g = torch.Generator(device="cuda")
    g.manual_seed(NB)
    q, k, v = (torch.randn((n, NB * 128, 128), generator=g, device="cuda").bfloat16() * 2
               for n in (hq, 1, 1))
    print(f"forward lists hq={hq} NB={NB} tau={tau} causal={causal}", flush=True)
    _, _, views = X.xattn_forward(q, k, v, causal=causal, stride=16, tau=tau)
    sc = X.xattn_score(q, k, causal=causal, stride=16)
    idx, cnt = X.xattn_select(sc, X.make_dims(q, k, causal), tau)
    torch.cuda.synchronize()
    assert torch.equal(views["scores"], sc) and torch.equal(views["cnt"], cnt)
    kept = torch.arange(NB, device="cuda") < cnt[..., None]
    assert torch.equal(views["idx"][kept], idx[kept])


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("hq,NB,stride", [(1, 9, 1), (2, 33, 1), (1, 129, 1), (1, 64, 2),
                                          (3, 65, 2), (2, 257, 2), (1, 65, 4)])
def test_forward_lists_at_small_strides(hq, NB, stride, causal):
    """The same where the finalisation keeps several loads of a row's stats in flight."""
    g = torch.Generator(device="cuda")
    g.manual_seed(NB)
    q, k, v = (torch.randn((n, NB * 128, 128), generator=g, device="cuda").bfloat16() * 2
               for n in (hq, 1, 1))
    print(f"forward lists hq={hq} NB={NB} stride={stride} causal={causal}", flush=True)
    _, _, views = X.xattn_forward(q, k, v, causal=causal, stride=stride, tau=0.9)
    sc = X.xattn_score(q, k, causal=causal, stride=stride)
    idx, cnt = X.xattn_select(sc, X.make_dims(q, k, causal), 0.9)
    torch.cuda.synchronize()
    assert torch.allclose(sc.sum(-1), torch.ones_like(sc[..., 0]), atol=1e-4)
    assert torch.equal(views["scores"], sc) and torch.equal(views["cnt"], cnt)
    kept = torch.arange(NB, device="cuda") < cnt[..., None]
    assert torch.equal(views["idx"][kept], idx[kept])
