"""The calls whose speed is measured: what a prefill engine, a video-diffusion
sampler or a threshold calibration has this library do, through its public
entry points, over the range of sizes that they meet.

A case is a dict of plain values. `op` names the call:

  forward    score -> select -> attention, a layer's prefill (`call`: the entry
             point: "forward" with a kept workspace, "noalloc", "scheduled")
  score      the block scores alone (`pattern`: antidiagonal or diagonal)
  select     the block lists from scores (`rule`: one threshold, one per head,
             Top-K, Top-Ratio)
  sparse     attention over given lists
  dense      attention over every block (`call`: "dense", or "scheduled" for a
             sampler's warm-up steps)
  error      a head's output error against the dense output

`blocks` counts 128-token blocks, so odd counts are the ragged sizes: a
reduced row or column tile of the scoring is then partly empty.
"""
from __future__ import annotations

import math

import torch

import paper_2503_16428_amd as X

BLOCK = 128
DIM = 128


def listed():
    return [
        # One head of a 4K-token prompt: the smallest call, as of a layer split over many ranks.
        dict(name="forward_4k_1head", op="forward", call="forward", batch=1, hq=1, hkv=1,
             blocks=32, causal=True, stride=8, tau=0.9, kind="clustered"),
        # Two 4736-token prompts of a small GQA model, an odd number of blocks.
        dict(name="forward_4736_batch2", op="forward", call="forward", batch=2, hq=8, hkv=2,
             blocks=37, causal=True, stride=16, tau=0.9, kind="clustered"),
        # A whole 8K-token layer in a server that allocates nothing.
        dict(name="forward_8k_noalloc", op="forward", call="noalloc", batch=1, hq=32, hkv=8,
             blocks=64, causal=True, stride=8, tau=0.9, kind="clustered"),
        # A whole 32K-token layer.
        dict(name="forward_32k", op="forward", call="forward", batch=1, hq=32, hkv=8,
             blocks=256, causal=True, stride=8, tau=0.9, kind="clustered"),
        # A whole 128K-token layer, the benchmark's own size.
        dict(name="forward_128k", op="forward", call="forward", batch=1, hq=32, hkv=8,
             blocks=1024, causal=True, stride=16, tau=0.9, kind="local"),
        # A 115,200-token video layer (30 x 60 x 64), bidirectional, past the warm-up steps.
        dict(name="forward_video_115200", op="forward", call="scheduled", batch=1, hq=24, hkv=24,
             blocks=900, causal=False, stride=16, tau=0.9, kind="video"),
        # The finest stride of the threshold x stride sweep at 64K tokens.
        dict(name="score_64k_stride4", op="score", pattern="antidiagonal", batch=1, hq=32, hkv=8,
             blocks=512, causal=True, stride=4, kind="clustered"),
        # The lists of a 64K-token layer, each head with its own calibrated threshold.
        dict(name="select_64k_heads", op="select", rule="heads", batch=1, hq=32, hkv=8,
             blocks=512, causal=True, value=0.9),
        # Attention over lists that the caller made, 16K tokens, query groups of 7.
        dict(name="sparse_16k_group7", op="sparse", batch=1, hq=28, hkv=4, blocks=125, causal=True,
             keep=0.25, kind="clustered"),
        # The dense reference of a 16K-token layer.
        dict(name="dense_16k", op="dense", call="dense", batch=1, hq=32, hkv=8, blocks=128,
             causal=True, kind="clustered"),
        # A warm-up step of a short video (15 x 30 x 32 tokens), dense and bidirectional.
        dict(name="dense_video_14464", op="dense", call="scheduled", batch=1, hq=24, hkv=24,
             blocks=113, causal=False, kind="clustered"),
        # One column of the calibration's error table on a 32K-token layer.
        dict(name="error_32k", op="error", batch=1, hq=32, hkv=8, blocks=256, causal=True),
    ]


HEADS = [(1, 1), (2, 1), (4, 4), (8, 1), (8, 2), (8, 8), (12, 4), (16, 2), (24, 24), (28, 4),
         (32, 8), (32, 32)]


def draw(rng):
    """A case of the same ranges: log-spread lengths, any head layout, stride and rule."""
    op = rng.choice(["forward"] * 6 + ["score"] * 3 + ["select"] * 2 + ["sparse"] * 2 +
                    ["dense"] * 2 + ["error"])
    hq, hkv = rng.choice(HEADS)
    case = dict(op=op, batch=rng.choice([1, 1, 1, 2, 3]), hq=hq, hkv=hkv,
                blocks=int(round(math.exp(rng.uniform(math.log(8), math.log(1024))))),
                causal=rng.random() < 0.7)
    if op in ("forward", "score"):
        case["stride"] = rng.choice([1, 2, 4, 4, 8, 8, 8, 8, 16, 16, 16, 16, 32, 64])
    if op == "forward":
        case["tau"] = rng.choice([0.8, 0.9, 0.9, 0.95, 1.0])
        case["call"] = rng.choice(["forward", "forward", "scheduled", "noalloc"])
        case["kind"] = rng.choice(["clustered", "clustered", "local", "video"])
    elif op == "score":
        case["pattern"] = rng.choice(["antidiagonal", "antidiagonal", "diagonal"])
        case["kind"] = rng.choice(["clustered", "local", "video"])
    elif op == "select":
        case["rule"] = rng.choice(["one", "one", "heads", "topk", "ratio"])
        case["value"] = (rng.randint(1, case["blocks"]) if case["rule"] == "topk"
                         else round(rng.uniform(0.05, 0.98), 3))
    elif op == "sparse":
        case["keep"] = round(rng.uniform(0.03, 0.5), 3)
        case["kind"] = "clustered"
    elif op == "dense":
        case["call"] = rng.choice(["dense", "scheduled"])
        case["kind"] = "clustered"
    while _cost(case) > 1.0:
        case["blocks"] = max(8, case["blocks"] * 4 // 5)
        if case["blocks"] == 8:
            case["batch"] = 1
    if case.get("rule") == "topk":
        case["value"] = min(case["value"], case["blocks"])
    return case


def _cost(case):
    """A rough share of the most that a case may cost."""
    flops = sum(_flops(case))
    if case.get("stride", 8) < 4:  # many reduced rows: the softmax outweighs the products
        flops *= 8 / case["stride"]
    size = case["blocks"] * BLOCK * DIM * case["batch"] * case["hq"] * 2  # bytes of q
    part = 0
    if "stride" in case:
        part = case["batch"] * case["hq"] * case["blocks"] ** 2 * 4 * BLOCK / case["stride"]
        if case["causal"]:
            part /= 2
    if case.get("call") == "noalloc" and _noalloc_bytes(case) > 60 << 20:
        return 2.0
    return max(flops / 8e12, size / 1.1e9, part / 2e9)


def _noalloc_bytes(case):
    heads = case["batch"] * case["hq"]
    square = case["blocks"] ** 2
    rows = BLOCK // case["stride"]
    stats = 8 * (case["blocks"] * rows) * (case["blocks"] * rows / 128 + 1)
    return heads * (8 * square + 4 * case["blocks"] + 4 * square * rows + stats)


def _share(case):
    """The share of the candidate blocks that attention reads: given, all, or about what a
    threshold keeps of these inputs (54 % at 32 blocks, 15 % at 256, 4-8 % from 512)."""
    if case["op"] == "dense":
        return 1.0
    if case["op"] == "sparse":
        return case["keep"]
    if case["tau"] >= 1.0:
        return 1.0
    return min(1.0, 20.0 / case["blocks"] ** 0.9) * (0.6 + 4.0 * (case["tau"] - 0.8))


def _flops(case):
    """(scoring, attention) operations of one pass, the causal half counted."""
    heads = case["batch"] * case["hq"]
    seq = case["blocks"] * BLOCK
    half = 0.5 if case["causal"] else 1.0
    score = attn = 0.0
    if case["op"] in ("forward", "score"):
        score = 2.0 * seq * seq / case["stride"] * DIM * heads * half
    if case["op"] in ("forward", "sparse", "dense"):
        attn = 4.0 * seq * seq * DIM * heads * half * _share(case)
    return score, attn


def work(case):
    heads, kv = case["batch"] * case["hq"], case["batch"] * case["hkv"]
    seq = case["blocks"] * BLOCK
    q, k = heads * seq * DIM * 2, kv * seq * DIM * 2
    half = 0.5 if case["causal"] else 1.0
    square = heads * case["blocks"] ** 2
    op = case["op"]
    if op == "select":
        # candidates read, every list entry written (the unused ones hold -1)
        return {"bytes": 4 * square * half + 4 * square + 4 * heads * case["blocks"], "flops": 0}
    if op == "error":
        return {"bytes": 2 * q + 8 * heads, "flops": 0}
    flops = sum(_flops(case))
    if op == "score":
        return {"bytes": q + k + 4 * square, "flops": flops}
    lse = 4 * heads * seq
    lists = 4 * square * half * _share(case) if op == "sparse" else 0
    return {"bytes": 2 * q + 2 * k + lse + lists, "flops": flops}


def _normal(shape, gen):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)


def _field(heads, seq, gen):
    """A smooth positional field, unit variance: 16 sinusoids over three axes."""
    pos = torch.arange(seq, device="cuda", dtype=torch.float32)
    cols = max(1, int(round(seq ** (1 / 3))))
    axes = torch.stack([(pos // (cols * cols)) / cols, (pos // cols % cols) / cols,
                        (pos % cols) / cols], 1)
    freq = 4.0 * torch.rand((heads, 3, 16), generator=gen, device="cuda")
    phase = 2 * math.pi * torch.rand((heads, 1, 16), generator=gen, device="cuda")
    amp = _normal((heads, 16, DIM), gen)
    out = []
    for h in range(heads):
        out.append(torch.sin(2 * math.pi * (axes @ freq[h]) + phase[h]) @ amp[h] / math.sqrt(8.0))
    return out


def _qkv(case, gen):
    """q, k, v of one layer in bfloat16: queries and keys around shared centres (64 a key head),
    the keys leaning on their predecessors ("local"), or noise on a smooth field ("video")."""
    b, hq, hkv, seq = case["batch"], case["hq"], case["hkv"], case["blocks"] * BLOCK
    group = hq // hkv
    q = torch.empty((b * hq, seq, DIM), dtype=torch.bfloat16, device="cuda")
    k = torch.empty((b * hkv, seq, DIM), dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    if case["kind"] == "video":
        fields = _field(b * hkv, seq, gen)
        for g in range(b * hkv):
            k[g] = _normal((seq, DIM), gen) + 2 * fields[g]
            for h in range(g * group, (g + 1) * group):
                q[h] = _normal((seq, DIM), gen) + 2 * fields[g]
            v[g] = _normal((seq, DIM), gen)
    else:
        def rows(centres):
            at = torch.randint(0, 64, (seq,), generator=gen, device="cuda")
            return centres[at] + _normal((seq, DIM), gen)

        for g in range(b * hkv):
            centres = 3 * _normal((64, DIM), gen)
            x = rows(centres)
            if case["kind"] == "local":
                x0 = x
                x = x0.clone()
                for back in range(1, 5):
                    x[4:] += 0.125 * x0[4 - back:seq - back]
            k[g] = x
            for h in range(g * group, (g + 1) * group):
                q[h] = rows(centres)
            v[g] = _normal((seq, DIM), gen)
    return q.view(b, hq, seq, DIM), k.view(b, hkv, seq, DIM), v.view(b, hkv, seq, DIM)


def _scores(case, gen):
    """Score rows as the scoring gives them: a few large masses, each row adding up to 1."""
    heads, nb = case["batch"] * case["hq"], case["blocks"]
    s = torch.rand((heads, nb, nb), generator=gen, device="cuda") ** 3.3
    if case["causal"]:
        s = torch.tril(s)
    return s / s.sum(-1, keepdim=True)


def _lists(case, gen):
    """Ascending lists with the first and the last candidate in each, about `keep` of the rest."""
    heads, nb = case["batch"] * case["hq"], case["blocks"]
    r = torch.rand((heads, nb, nb), generator=gen, device="cuda") < case["keep"]
    j = torch.arange(nb, device="cuda", dtype=torch.int32)
    r[:, :, 0] = True
    if case["causal"]:
        r &= j[None, :] <= j[:, None]
        r |= j[None, :] == j[:, None]
    else:
        r[:, :, nb - 1] = True
    idx = torch.where(r, j.expand_as(r), nb).sort(-1).values
    return torch.where(idx < nb, idx, -1).int().contiguous(), r.sum(-1).int().contiguous()


def _per_head(case):
    hq, v = case["hq"], case["value"]
    if case["rule"] == "heads":
        return [min(1.0, v * (0.9 + 0.1 * h / max(1, hq - 1))) for h in range(hq)]
    if case["rule"] == "topk":
        return [max(1, int(v) - h % 3) for h in range(hq)]
    return [v * (0.8 + 0.2 * h / max(1, hq - 1)) for h in range(hq)]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    heads, seq = case["batch"] * case["hq"], case["blocks"] * BLOCK
    s = {"case": case, "dims": X.Dims(case["batch"], case["hq"], case["hkv"], seq, DIM,
                                      int(case["causal"]))}
    op = case["op"]
    if op in ("forward", "score", "sparse", "dense"):
        s["q"], s["k"], s["v"] = _qkv(case, gen)
    if op in ("forward", "sparse", "dense"):
        s["o"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((heads, seq), dtype=torch.float32, device="cuda")
    if op == "forward" and case["call"] != "noalloc":
        s["ws"] = torch.empty(X.forward_workspace_size(s["dims"], BLOCK, case["stride"]),
                              dtype=torch.uint8, device="cuda")
    if op == "score":
        s["ws"] = torch.empty(X.score_workspace_size(s["dims"], BLOCK, case["stride"]),
                              dtype=torch.uint8, device="cuda")
        s["scores"] = torch.empty((heads, case["blocks"], case["blocks"]), dtype=torch.float32,
                                  device="cuda")
    if op == "select":
        s["scores"] = _scores(case, gen)
    if op == "sparse":
        s["idx"], s["cnt"] = _lists(case, gen)
    if op == "error":
        shape = (case["batch"], case["hq"], seq, DIM)
        ref = _normal(shape, gen)
        s["ref"] = ref.bfloat16()
        s["o"] = (ref + 0.1 * _normal(shape, gen)).bfloat16()
    return s


def run(s):
    c, op = s["case"], s["case"]["op"]
    if op == "forward":
        if c["call"] == "noalloc":
            o, lse = X.xattn_forward_noalloc(s["q"], s["k"], s["v"], s["o"], s["lse"], c["causal"],
                                             BLOCK, c["stride"], c["tau"])
            return {"o": o, "lse": lse}
        if c["call"] == "scheduled":
            o, lse = X.xattn_forward_scheduled(s["q"], s["k"], s["v"], 5, 5, c["causal"], BLOCK,
                                               c["stride"], c["tau"], s["o"], s["lse"], s["ws"])
            return {"o": o, "lse": lse}
        o, lse, views = X.xattn_forward(s["q"], s["k"], s["v"], c["causal"], BLOCK, c["stride"],
                                        c["tau"], s["o"], s["lse"], s["ws"])
        return {"o": o, "lse": lse, "scores": views["scores"], "cnt": views["cnt"]}
    if op == "score":
        if c["pattern"] == "diagonal":
            return {"scores": X.xattn_score_pattern(s["q"], s["k"], c["causal"], BLOCK,
                                                    c["stride"], list(range(c["stride"])),
                                                    s["scores"], s["ws"])}
        return {"scores": X.xattn_score(s["q"], s["k"], c["causal"], BLOCK, c["stride"],
                                        s["scores"], s["ws"])}
    if op == "select":
        if c["rule"] == "one":
            idx, cnt = X.xattn_select(s["scores"], s["dims"], c["value"])
        elif c["rule"] == "heads":
            idx, cnt = X.xattn_select_heads(s["scores"], s["dims"], _per_head(c))
        elif c["rule"] == "topk":
            idx, cnt = X.xattn_select_topk(s["scores"], s["dims"], _per_head(c))
        else:
            idx, cnt = X.xattn_select_ratio(s["scores"], s["dims"], _per_head(c))
        return {"idx": idx, "cnt": cnt}
    if op == "sparse":
        o, lse = X.xattn_block_sparse_attn(s["q"], s["k"], s["v"], s["idx"], s["cnt"], c["causal"],
                                           BLOCK, s["o"], s["lse"])
        return {"o": o, "lse": lse}
    if op == "dense":
        if c["call"] == "scheduled":
            o, lse = X.xattn_forward_scheduled(s["q"], s["k"], s["v"], 0, 5, c["causal"], BLOCK,
                                               16, 0.9, s["o"], s["lse"])
        else:
            o, lse = X.xattn_dense_attn(s["q"], s["k"], s["v"], c["causal"], s["o"], s["lse"])
        return {"o": o, "lse": lse}
    return {"err": X.head_error(s["o"], s["ref"], c["causal"])}


def tolerance(case):
    op = case["op"]
    if op == "select":
        return "exact"
    if op == "error":  # 64-bit sums in another order
        return {"rel": 1e-12}
    if op == "score":  # 32-bit sums of up to 8192 products, then exponentials: 2.1e-6 seen
        return {"rel": 1e-5}
    if op in ("sparse", "dense"):  # probabilities and outputs in bfloat16: 0.0022 seen
        return {"rel": 1e-2, "max": 0.1}
    # As for attention; besides, where a row's cumulative mass meets the threshold to within the
    # 32-bit scores' own rounding a block more or less is kept, and that row's outputs differ.
    return {"rel": 1e-2, "max": 0.99, "differ": 2e-3}


def _exact_scores(q, k, case, pairing):
    b, hq, seq, _ = q.shape
    group, s, nb = hq // k.shape[1], case["stride"], case["blocks"]
    nr, per = seq // s, BLOCK // s
    qs, ks = q.reshape(b * hq, seq, DIM), k.reshape(-1, seq, DIM)
    out = torch.zeros((b * hq, nb, nb), dtype=torch.float64, device=q.device)
    col = torch.arange(nr, device=q.device)
    step = max(1, min(nb, (1 << 27) // (nr * per))) * per
    for h in range(b * hq):
        kt = ks[h // group].double().view(nr, s * DIM).t().contiguous()
        qt = qs[h].view(nr, s, DIM)[:, pairing].reshape(nr, s * DIM)
        for r0 in range(0, nr, step):
            r1 = min(nr, r0 + step)
            c1 = r1 if case["causal"] else nr
            x = (qt[r0:r1].double() @ kt[:, :c1]) / (s * math.sqrt(DIM))
            if case["causal"]:
                x.masked_fill_(col[None, :c1] > col[r0:r1, None], -math.inf)
            p = torch.softmax(x, -1).view((r1 - r0) // per, per, c1 // per, per).sum((1, 3)) / per
            out[h, r0 // per:r1 // per, :c1 // per] = p
    return out


def _exact_select(scores, tau, causal):
    """Per row the kept blocks, ascending, and their number."""
    heads, nb, _ = scores.shape
    j = torch.arange(nb, device=scores.device)
    cand = (j[None, :] <= j[:, None]) if causal else torch.ones((nb, nb), dtype=torch.bool,
                                                                device=scores.device)
    if tau >= 1.0:
        keep = cand.expand(heads, nb, nb)
    else:
        u = (scores.clamp(0, 1) * 4294967296.0).floor().long()
        u = torch.where(cand, u, -1)
        order = u.sort(dim=-1, descending=True, stable=True)
        mass = order.values.clamp(min=0)
        total = mass.sum(-1, keepdim=True)
        tau32 = float(torch.tensor(tau, dtype=torch.float32))
        want = (tau32 * total.double()).ceil().long()
        before = mass.cumsum(-1) - mass
        keep = torch.zeros_like(u, dtype=torch.bool).scatter_(-1, order.indices, before < want)
        keep &= cand
    idx = torch.where(keep, j.expand_as(keep), nb).sort(-1).values
    return idx, keep.sum(-1)


def _exact_attention(q, k, v, idx, cnt, causal):
    b, hq, seq, _ = q.shape
    group, nb = hq // k.shape[1], seq // BLOCK
    qs = q.reshape(b * hq, nb, BLOCK, DIM)
    ks, vs = k.reshape(-1, nb, BLOCK, DIM), v.reshape(-1, nb, BLOCK, DIM)
    o = torch.empty((b * hq, nb, BLOCK, DIM), dtype=torch.float64, device=q.device)
    lse = torch.empty((b * hq, nb, BLOCK), dtype=torch.float64, device=q.device)
    at = torch.arange(BLOCK, device=q.device)
    counts = cnt.cpu().tolist()
    for h in range(b * hq):
        kd, vd, qd = ks[h // group].double(), vs[h // group].double(), qs[h].double()
        for i in range(nb):
            j = idx[h, i, :counts[h][i]].long()
            x = qd[i] @ kd[j].view(-1, DIM).t() / math.sqrt(DIM)
            if causal:
                key = (j[:, None] * BLOCK + at).view(-1)
                x.masked_fill_(key[None, :] > (i * BLOCK + at)[:, None], -math.inf)
            lse[h, i] = torch.logsumexp(x, -1)
            o[h, i] = torch.exp(x - lse[h, i][:, None]) @ vd[j].view(-1, DIM)
    return o.view(q.shape), lse.view(b * hq, seq)


def exact(case, seed):
    """What run() returns, in 64 bits and plain torch; the lists of a forward pass come from the
    64-bit scores."""
    op = case["op"]
    if op == "select" or sum(_flops(case)) > 3e13:
        return None
    if case["batch"] * case["hq"] * case["blocks"] > 100_000:
        return None
    s = prepare(case, seed)
    if op == "error":
        o, ref = (s[n].flatten(0, 1).double() for n in ("o", "ref"))
        return {"err": ((o - ref) ** 2).sum((1, 2)) / (ref ** 2).sum((1, 2))}
    nb, heads = case["blocks"], case["batch"] * case["hq"]
    scores = None
    if op in ("forward", "score"):
        st = case["stride"]
        diagonal = case.get("pattern") == "diagonal"
        pairing = list(range(st)) if diagonal else list(range(st - 1, -1, -1))
        scores = _exact_scores(s["q"], s["k"], case, pairing)
        if op == "score":
            return {"scores": scores}
        idx, cnt = _exact_select(scores, case["tau"], case["causal"])
    elif op == "sparse":
        idx, cnt = s["idx"], s["cnt"]
    else:
        idx = torch.arange(nb, device="cuda").expand(heads, nb, nb)
        cnt = (torch.arange(1, nb + 1, device="cuda") if case["causal"]
               else torch.full((nb,), nb, device="cuda")).expand(heads, nb)
    o, lse = _exact_attention(s["q"], s["k"], s["v"], idx, cnt, case["causal"])
    if op == "forward" and case["call"] == "forward":
        return {"o": o, "lse": lse, "scores": scores, "cnt": None}
    return {"o": o, "lse": lse}
