"""The calls this library is timed on: whole prefill layers and their stages.

Every case is a dict of plain values.  ``kind`` says which public entry
points one pass calls:

  layer    ``prefill``: metadata, scores and selection, route, attention over lists
  fused    ``prefill_fused``: the same layer with the selection inside the attention kernel
  select   ``ugbs_score_select`` alone, on metadata in hand
  attend   ``ugbs_attend`` alone, on routed lists in hand
  rows     ``ugbs_select_rows`` then ``ugbs_attend_bitmap``
  bai      the Appendix D diagnostics: ``ugbs_noise_scale``, ``ugbs_bai_tiles``, ``ugbs_bai_heads``

Inputs are drawn on the GPU from the seed with the distributions of
``paper_2607_07724_amd/synth.py``: Gaussian queries and values, keys with a
Gaussian offset per block ("offset") or from 64 cluster centres ("mixture"),
rows RMS-normalised where the model normalises queries and keys (d 256).
Lists, metadata and flags that a pass takes as given come from plain torch,
not from the library, so every version of it gets the same ones.
"""
from __future__ import annotations

import math

import torch

import paper_2607_07724_amd as ugbs

BLK = 64
HEADS = [(4, 1), (8, 2), (28, 4), (32, 8), (16, 2), (6, 3), (3, 3)]


def _case(kind, B, H, Hkv, N, d, k, q, quest, rho=2, **more):
    return dict(kind=kind, B=B, H=H, Hkv=Hkv, N=N, d=d, k=k, q=q, quest=quest, rho=rho, **more)


def listed():
    return [
        # the smallest layer (4 query / 1 kv head, d 64, 1K): launches and latency
        dict(_case("layer", 1, 4, 1, 1024, 64, 4, 0.25, False), name="layer_1k_d64"),
        # a short prompt on the Mistral-Nemo attention shape
        dict(_case("layer", 1, 32, 8, 4096, 128, 16, 0.1, True), name="layer_4k"),
        # the Qwen2.5-7B-1M attention shape at 32K, K-mean scores
        dict(_case("layer", 1, 28, 4, 32768, 128, 32, 0.1, False), name="layer_32k"),
        # the Mistral-Nemo attention shape at 128K, Quest scores: the benchmark's layer
        dict(_case("layer", 1, 32, 8, 131072, 128, 64, 0.1, True), name="layer_128k"),
        # two sequences of an odd number of blocks (141), selection inside the
        # attention kernel, the paper's operating point k 33, q 0.4
        dict(_case("fused", 2, 28, 4, 9024, 128, 33, 0.4, True), name="fused_9k_b2"),
        # scores and sorted selection at 128K, Quest
        dict(_case("select", 1, 32, 8, 131072, 128, 64, 0.1, True), name="select_128k"),
        # the same stage with K-mean scores on an odd length (1021 blocks)
        dict(_case("select", 1, 28, 4, 65344, 128, 33, 0.4, False), name="select_64k_kmean"),
        # attention over routed lists, Qwen2.5-7B-1M shape at 64K
        dict(_case("attend", 1, 28, 4, 65536, 128, 64, 0.1, True), name="attend_64k"),
        # attention of the Qwen3.6 full-attention layers (d 256, 8 query heads per kv head)
        dict(_case("attend", 1, 16, 2, 65536, 256, 33, 0.4, False), name="attend_64k_d256"),
        # attention at d 64 with rho 4 on an odd length (253 blocks)
        dict(_case("attend", 1, 16, 4, 16192, 64, 16, 0.25, True, rho=4), name="attend_16k_d64"),
        # per-row selection into bitmaps and the attention over them, 32K
        dict(_case("rows", 1, 28, 4, 32768, 128, 32, 0.1, True), name="rows_32k"),
        # the diagnostics of one layer at 32K with 256 Monte Carlo samples
        dict(_case("bai", 1, 28, 4, 32768, 128, 32, 0.1, False, samples=256), name="bai_32k"),
    ]


def draw(rng):
    def blocks(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["layer", "layer", "fused", "select", "attend", "attend", "rows", "bai"])
    H, Hkv = rng.choice(HEADS)
    d = rng.choice([64, 128, 128, 128, 256])
    most = {"layer": 1024, "fused": 1024, "select": 2048, "attend": 1024, "rows": 384, "bai": 768}[kind]
    nb = blocks(16, most)
    B = 2 if nb <= most // 2 and rng.random() < 0.25 else 1
    # budgets as used: a fraction of the visible blocks, at least 4, at most 64
    k = max(4, min(64, int(nb * rng.uniform(0.03, 0.3))))
    rho = rng.choice([2, 2, 2, 3, 4])
    q = rng.choice([0.05, 0.1, 0.25, 0.4])
    c = _case(kind, B, H, Hkv, BLK * nb, d, k, q, rng.random() < 0.5, rho=rho)
    if kind == "bai":
        c["samples"] = rng.choice([64, 200, 256])
    return c


# ------------------------------------------------------------------ inputs

def _problem(c):
    return ugbs.Problem.make(c["B"], c["H"], c["Hkv"], c["N"], c["d"], c["k"], c["q"],
                             ugbs.QUEST if c["quest"] else ugbs.KMEAN, rho=c["rho"])


def _norm(x):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6)


def _qkv(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, Hkv, N, d = c["B"], c["H"], c["Hkv"], c["N"], c["d"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    Q = torch.empty((B, H, N, d), dtype=torch.bfloat16, device="cuda")
    K = torch.empty((B, Hkv, N, d), dtype=torch.bfloat16, device="cuda")
    V = torch.empty_like(K)
    for b in range(B):
        for h in range(H):
            x = normal(N, d)
            Q[b, h] = _norm(x) if d == 256 else x
        for h in range(Hkv):
            if c["quest"]:    # keys around 64 cluster centres
                at = torch.randint(0, 64, (N,), generator=g, device="cuda")
                x = normal(64, d)[at] + 0.3 * normal(N, d)
            else:             # a common offset per block
                x = normal(N, d) + 0.5 * normal(N // BLK, d).repeat_interleave(BLK, 0)
            K[b, h] = _norm(x) if d == 256 else x
            V[b, h] = normal(N, d)
    return Q, K, V, g


def _meta(c, K):
    blocks = K.view(c["B"], c["Hkv"], c["N"] // BLK, BLK, c["d"])
    if not c["quest"]:
        return blocks.double().mean(3).to(torch.bfloat16).unsqueeze(-1).contiguous()
    return torch.stack([blocks.amin(3), blocks.amax(3)], -1).contiguous()


def _row_scores(c, Qh, meta_h, dtype):
    """[N, N_B] scores of one head's query rows against one kv head's blocks."""
    m = meta_h.to(dtype)
    q = Qh.to(dtype)
    if not c["quest"]:
        return q @ m[..., 0].t().contiguous()
    both = torch.cat([m[..., 0], m[..., 1]], 1).t().contiguous()
    return torch.cat([q.clamp(max=0), q.clamp(min=0)], 1) @ both


def _tile_scores(c, Q, meta, dtype, out=torch.float32):
    B, H, N = c["B"], c["H"], c["N"]
    T = N // BLK
    S = torch.empty((B, H, T, T), dtype=out, device="cuda")
    for b in range(B):
        for h in range(H):
            kvh = h // (H // c["Hkv"])
            for n0 in range(0, N, 32768):
                s = _row_scores(c, Q[b, h, n0:n0 + 32768], meta[b, kvh], dtype)
                S[b, h, n0 // BLK:(n0 + s.shape[0]) // BLK] = s.view(-1, BLK, T).amax(1)
    blk = torch.arange(T, device="cuda")
    inside = (blk[None, :] >= 1) & (blk[None, :] < blk[:, None])      # candidates 1..t-1 of tile t
    return S.masked_fill_(~inside, -math.inf)


def _lists(c, S, trigger):
    """kv_idx [B, H, T, rho k]: sink, own block, then the best candidates."""
    T, W, k = c["N"] // BLK, c["rho"] * c["k"], c["k"]
    n = min(W - 2, T)
    top = torch.topk(S, n, dim=-1)
    kv = torch.full(S.shape[:3] + (W,), T, dtype=torch.int32, device="cuda")
    kv[..., 2:2 + n] = torch.where(top.values == -math.inf, T, top.indices).int()
    kv[..., 0] = 0
    kv[..., 1] = torch.arange(T, device="cuda", dtype=torch.int32)
    kv[:, :, 0, 1] = T
    cut = (trigger == 0)[:, None, :, None] & (torch.arange(W, device="cuda") >= k)
    return kv.masked_fill_(cut, T)


def _flags(c, g):
    """Trigger flags on about a share q of the tiles that keep fewer blocks than they see."""
    T = c["N"] // BLK
    f = torch.rand((c["B"], T), generator=g, device="cuda") < c["q"]
    return (f & (torch.arange(T, device="cuda") > c["k"] - 1)).to(torch.uint8)


def prepare(case, seed):
    c, p = case, _problem(case)
    Q, K, V, g = _qkv(c, seed)
    st = dict(kind=c["kind"], p=p, Q=Q, K=K, V=V)
    B, H, T = c["B"], c["H"], p.T
    if c["kind"] in ("layer", "fused"):
        st["bufs"] = ugbs.Buffers(p)
        st["O"] = torch.empty_like(Q)
        return st
    meta = _meta(c, K)
    if c["kind"] == "select":
        st["meta"] = meta
        st["idx"] = torch.empty((B, H, T, p.W), dtype=torch.int32, device="cuda")
        st["sigma"] = torch.empty((B, H, T), dtype=torch.float32, device="cuda")
        st["ws"] = torch.empty((max(256, ugbs.ugbs_workspace_bytes(p)),), dtype=torch.uint8, device="cuda")
        del st["K"], st["V"]
    elif c["kind"] == "attend":
        st["kv_idx"] = _lists(c, _tile_scores(c, Q, meta, torch.bfloat16), _flags(c, g))
        st["O"] = torch.empty_like(Q)
    elif c["kind"] == "rows":
        st["meta"] = meta
        st["trigger"] = _flags(c, g)
        st["bitmap"] = torch.empty((B, H, T, ugbs.bitmap_words(p)), dtype=torch.int32, device="cuda")
        st["O"] = torch.empty_like(Q)
    else:
        st["meta"] = meta
        st["scores"] = _tile_scores(c, Q, meta, torch.bfloat16)
        st["z"] = torch.randn((p.NB, c["samples"]), generator=g, device="cuda")
        st["rough"] = torch.empty((B, H, T), dtype=torch.float64, device="cuda")
        st["tau"] = torch.empty((B, H), dtype=torch.float32, device="cuda")
        st["tiles"] = torch.empty((B, H, T, ugbs.BAI_TILE_BYTES), dtype=torch.uint8, device="cuda")
        st["heads"] = torch.empty((B, H, ugbs.BAI_HEAD_BYTES), dtype=torch.uint8, device="cuda")
        del st["K"], st["V"]
    return st


def run(st):
    p, kind = st["p"], st["kind"]
    if kind in ("layer", "fused"):
        b = st["bufs"]
        (ugbs.prefill if kind == "layer" else ugbs.prefill_fused)(p, st["Q"], st["K"], st["V"], st["O"], b)
        out = dict(O=st["O"], sigma=b.sigma, sigma_bar=b.sigma_bar, trigger=b.trigger)
        if kind == "layer":
            out["kv_idx"] = b.kv_idx
        return out
    if kind == "select":
        ugbs.ugbs_score_select(p, st["Q"], st["meta"], st["idx"], st["sigma"], workspace=st["ws"])
        return dict(idx=st["idx"], sigma=st["sigma"])
    if kind == "attend":
        ugbs.ugbs_attend(p, st["Q"], st["K"], st["V"], st["kv_idx"], st["O"])
        return dict(O=st["O"])
    if kind == "rows":
        ugbs.ugbs_select_rows(p, st["trigger"], st["bitmap"], Q=st["Q"], meta=st["meta"])
        ugbs.ugbs_attend_bitmap(p, st["Q"], st["K"], st["V"], st["bitmap"], st["O"])
        return dict(O=st["O"], bitmap=st["bitmap"])
    ugbs.ugbs_noise_scale(p, st["Q"], st["meta"], st["rough"], st["tau"])
    ugbs.ugbs_bai_tiles(p, st["scores"], st["tiles"], tau=st["tau"], z=st["z"])
    ugbs.ugbs_bai_heads(p, st["tiles"], st["tau"], int(st["z"].shape[1]), st["heads"])
    # the records as numbers: five gaps and three counts per tile, counts and aggregates per head
    return dict(rough=st["rough"], tau=st["tau"],
                tile_gaps=st["tiles"].view(torch.float32)[..., :5], tile_counts=st["tiles"].view(torch.int32)[..., 5:],
                head_counts=st["heads"].view(torch.int32)[..., :2], head_values=st["heads"].view(torch.float64)[..., 2:])


# ------------------------------------------------------------------ work

def _candidates(c):
    T = c["N"] // BLK
    return [max(t - 1, 0) for t in range(T)]


def _pairs(c, kept):
    """(query row, key) pairs of one head over tiles that keep `kept[t]` blocks, the last one causal."""
    return sum((n - 1) * BLK * BLK + BLK * (BLK + 1) // 2 for n in kept)


def _kept(c):
    k, W, q = c["k"], c["rho"] * c["k"], c["q"]
    T = c["N"] // BLK
    if c["kind"] != "rows":
        return [min(t + 1, k) + q * max(0, min(t + 1, W) - k) for t in range(T)]
    # the union over a tile's 64 rows, which choose like about 14 independent
    # ones on these inputs (195 blocks a tile at 32K, k 32)
    def union(t, slots):
        n = max(t - 1, 0)
        return min(t + 1, 2) + n * (1 - (1 - min(slots - 2, n) / max(n, 1)) ** 14)

    return [(1 - q) * union(t, k) + q * union(t, W) for t in range(T)]


def work(case):
    c = case
    B, H, Hkv, N, d = c["B"], c["H"], c["Hkv"], c["N"], c["d"]
    T, W = N // BLK, c["rho"] * c["k"]
    cols = 2 if c["quest"] else 1
    q_b, kv_b, meta_b = 2 * B * H * N * d, 2 * B * Hkv * N * d, 2 * B * Hkv * T * d * cols
    lists_b = 4 * B * H * T * W
    # one multiply-add per channel, row and candidate: K-mean the mean, Quest the minimum or the maximum
    score_f = 2 * d * BLK * B * H * sum(_candidates(c))
    attend_f = 4 * d * B * H * _pairs(c, _kept(c))
    if c["kind"] == "layer":
        return dict(bytes=2 * q_b + 2 * kv_b + lists_b, flops=score_f + attend_f)
    if c["kind"] == "fused":
        return dict(bytes=2 * q_b + 2 * kv_b, flops=score_f + attend_f)
    if c["kind"] == "select":
        return dict(bytes=q_b + meta_b + lists_b, flops=score_f)
    if c["kind"] == "attend":
        return dict(bytes=2 * q_b + 2 * kv_b + lists_b, flops=attend_f)
    if c["kind"] == "rows":
        return dict(bytes=2 * q_b + 2 * kv_b + meta_b, flops=score_f + attend_f)
    # scores of the noise scale; one draw (multiply, add, compare) per candidate and sample
    mc_f = 3 * c["samples"] * B * H * sum(_candidates(c))
    return dict(bytes=q_b + meta_b + 4 * B * H * sum(_candidates(c)) + 4 * T * c["samples"], flops=score_f + mc_f)


# ------------------------------------------------------------------ accuracy

def tolerance(case):
    # About four times the distance to the 64-bit results.  Attention (bf16
    # probabilities and outputs): 2.3e-3, largest 0.06.  Layers: a score that
    # rounds differently swaps two nearly tied blocks of a row now and then,
    # which moves that tile's output by up to the block's whole weight: 3.2e-3,
    # largest 1.4.  Selection: sigma is a difference of fp32 scores over a
    # difference of them, 1.8e-5, largest 1.1e-4.
    if case["kind"] in ("layer", "fused"):
        return {"rel": 0.013, "max": 0.99, "differ": 0.005}
    if case["kind"] == "rows":
        return {"rel": 0.013, "max": 0.99, "differ": 0.01}
    if case["kind"] == "attend":
        return {"rel": 0.01, "max": 0.25}
    if case["kind"] == "select":
        return {"rel": 1e-4, "max": 1e-3, "differ": 0.002}
    return {"rel": 1e-5, "max": 4e-4, "differ": 0.001}


def _exact_select(c, S):
    """sigma [B, H, T] in 64 bits from the tile scores (-1: every visible block is kept)."""
    T, k = c["N"] // BLK, c["k"]
    top = torch.topk(S, min(k, T), dim=-1).values
    if top.shape[-1] < k:
        return torch.full(S.shape[:3], -1.0, dtype=torch.float64, device=S.device)
    m = k - 2                                              # tiles of the population have t >= k
    num, den = top[..., m - 1] - top[..., m], top[..., 0] - top[..., m]
    sigma = torch.where(den == 0, 0.0, num / den)
    return torch.where(torch.arange(T, device=S.device) - 1 > m, sigma, -1.0)


def _exact_route(c, sigma):
    T, k = c["N"] // BLK, c["k"]
    pop = torch.arange(T, device=sigma.device) - 1 > k - 2
    bar = torch.where(pop, sigma.mean(1), -1.0)
    n_trig = math.ceil(c["q"] * int(pop.sum()))
    flags = torch.zeros(bar.shape, dtype=torch.uint8, device=sigma.device)
    for b in range(c["B"]):
        if n_trig:
            tau = bar[b][pop].sort().values[n_trig - 1]
            flags[b] = (pop & (bar[b] <= tau)).to(torch.uint8)
    return bar, flags


def _exact_attend(c, Q, K, V, keep):
    """Softmax attention in 64 bits; keep(b, h) -> [T, N_B] truth values, blocks attended per tile."""
    B, H, N, d = c["B"], c["H"], c["N"], c["d"]
    O = torch.empty(Q.shape, dtype=torch.float32, device=Q.device)
    per = max(1, int(2 ** 27 // (BLK * N)))                # tiles a step: at most 1 GiB of logits
    for b in range(B):
        for h in range(H):
            kvh = h // (H // c["Hkv"])
            Kt, Vd = K[b, kvh].double().t().contiguous(), V[b, kvh].double()
            on = keep(b, h)
            for t0 in range(0, N // BLK, per):
                t1 = min(t0 + per, N // BLK)
                rows = torch.arange(BLK * t0, BLK * t1, device=Q.device)
                L = BLK * t1
                s = (Q[b, h, BLK * t0:L].double() @ Kt[:, :L]) / math.sqrt(d)
                mask = on[t0:t1, :t1].repeat_interleave(BLK, 1).repeat_interleave(BLK, 0)
                mask &= torch.arange(L, device=Q.device)[None, :] <= rows[:, None]
                s.masked_fill_(~mask, -math.inf)
                O[b, h, BLK * t0:L] = (torch.softmax(s, 1) @ Vd[:L]).float()
    return O


def _listed(kv, T):
    on = torch.zeros(kv.shape[:1] + (T + 1,), dtype=torch.bool, device=kv.device)
    return on.scatter_(1, kv.long(), True)[:, :T]


def exact(case, seed):
    c = case
    T = c["N"] // BLK
    if c["kind"] not in ("select", "bai") and c["B"] * c["H"] * c["N"] ** 2 * c["d"] > 2 ** 44:
        return None                                        # over 20 s
    st = prepare(case, seed)
    Q, kind = st["Q"], c["kind"]
    if kind == "attend":
        return dict(O=_exact_attend(c, Q, st["K"], st["V"], lambda b, h: _listed(st["kv_idx"][b, h], T)))
    meta = st["meta"] if "meta" in st else _meta(c, st["K"])
    if kind == "rows":
        def keep(b, h):
            on = torch.eye(T, dtype=torch.bool, device="cuda")
            on[:, 0] = True
            m = meta[b, h // (c["H"] // c["Hkv"])]
            for t0 in range(0, T, 128):
                t1 = min(t0 + 128, T)
                s = _row_scores(c, Q[b, h, BLK * t0:BLK * t1], m, torch.float64).view(t1 - t0, BLK, T)
                t = torch.arange(t0, t1, device="cuda")[:, None, None]
                blk = torch.arange(T, device="cuda")
                s = s.masked_fill((blk < 1) | (blk >= t), -math.inf)
                R = torch.where(st["trigger"][b, t0:t1] != 0, c["rho"] * c["k"], c["k"]).long() - 2
                top = torch.topk(s, min(T, c["rho"] * c["k"] - 2), dim=-1)
                ok = (torch.arange(top.values.shape[-1], device="cuda") < R[:, None, None]) & (top.values > -math.inf)
                hit = torch.zeros((t1 - t0, BLK, T), dtype=torch.bool, device="cuda")
                hit.scatter_(2, top.indices, ok)
                on[t0:t1] |= hit.any(1)
            return on
        return dict(O=_exact_attend(c, Q, st["K"], st["V"], keep), bitmap=None)
    if kind == "bai":
        B, H, N = c["B"], c["H"], c["N"]
        rough = torch.zeros((B, H, T), dtype=torch.float64, device="cuda")
        blk = torch.arange(T, device="cuda")
        for b in range(B):
            for h in range(H):
                s = _row_scores(c, Q[b, h], meta[b, h // (H // c["Hkv"])], torch.float64).view(T, BLK, T)
                sq = (s[:, 1:] - s[:, :-1]).square().sum(1)
                rough[b, h] = (sq * ((blk >= 1) & (blk < blk[:, None]))).sum(1)
        tau = (rough.sum(2) / (2 * 63 * ((T - 1) * (T - 2) // 2))).sqrt()
        return dict(rough=rough, tau=tau, tile_gaps=None, tile_counts=None, head_counts=None, head_values=None)
    S = _tile_scores(c, Q, meta, torch.float64, out=torch.float64)
    sigma = _exact_select(c, S)
    if kind == "select":
        return dict(idx=None, sigma=sigma)
    bar, flags = _exact_route(c, sigma)
    kv = _lists(c, S, flags)
    del S
    out = dict(O=_exact_attend(c, Q, st["K"], st["V"], lambda b, h: _listed(kv[b, h], T)), sigma=sigma, sigma_bar=bar,
               trigger=None)
    if kind == "layer":
        out["kv_idx"] = None
    return out
