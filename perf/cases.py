"""The workloads that the library's speed is measured on: listed sizes and a generator of more of the same ranges.

A case is a plain dict.  Its `kind` says which public entry points one pass calls:

  call    dr_block_scores -> dr_build_mask -> dr_sparse_attn_fwd: one attention layer of a video model
  attend  dr_sparse_attn_fwd alone, on a block mask that the program already has (a mask is often kept over several
          denoising steps), with the log-sum-exp
  mask    dr_build_mask alone, per-head masks from scores that the program already has
  tokens  dr_build_mask_tokens on kept token scores: one step of a search over thresholds
  proxy   proxy_eval.proxy_loss: the whole objective of the offline search at one configuration

Inputs are synthetic, made on the GPU from the seed: a random-Fourier-feature field over the (t, y, x) token grid plus
noise, so that logits fall off with distance in space and time as they do in video models; `blob` adds an object that
moves across the grid; `drift` is the search's own proxy task, features that forget their past frame by frame.
"""
from __future__ import annotations

import math

import torch

import paper_2604_20470_amd as dr
from paper_2604_20470_amd import proxy_eval

MODES = {"static": dr.MODE_STATIC, "dynamic": dr.MODE_DYNAMIC, "zscore": dr.MODE_ZSCORE, "uniform": dr.MODE_UNIFORM}


def _case(kind, B, H, d, Nf, Hg, Wg, Bs, dtype, recipe, mode, par, lam, fuse, kept):
    """`kept`: the share of block pairs that such a mask keeps, for the count of operations in work()."""
    return dict(kind=kind, B=B, H=H, d=d, Nf=Nf, Hg=Hg, Wg=Wg, Bs=Bs, dtype=dtype, recipe=recipe, mode=mode, par=par,
                lam=lam, fuse=fuse, kept=kept)


def listed():
    out = []

    def add(name, *a):
        out.append(dict(_case(*a), name=name))

    # The smallest call: 256 tokens in fp32, as a unit test or a toy model makes it.  Launches are all it costs.
    add("call_tiny_f32", "call", 1, 2, 64, 4, 8, 8, 64, "f32", "iid", "static", 0.5, 0.5, 2, 0.625)
    # A short low-resolution clip, 6144 tokens x 8 heads: fewer pieces of work than the chip has compute units.
    add("call_small", "call", 1, 8, 128, 8, 24, 32, 128, "bf16", "field", "static", 0.2, 0.5, 2, 0.406)
    # 480p, 21 latent frames, 40 heads, cumulative-mass rule: an ordinary layer.
    add("call_480p", "call", 1, 40, 128, 21, 30, 52, 128, "bf16", "field", "dynamic", 0.9, 0.3, 2, 0.30)
    # 720p, 21 latent frames, 40 heads, top-k at 85 % sparsity: the headline workload.
    add("call_720p", "call", 1, 40, 128, 21, 45, 80, 128, "bf16", "field", "static", 0.043, 0.5, 2, 0.1497)
    # 720p, 33 latent frames, 24 heads, an object in motion: the longest sequence at the large block size.
    add("call_720p_long", "call", 1, 24, 128, 33, 45, 80, 128, "bf16", "blob", "dynamic", 0.95, 0.7, 2, 0.222)
    # 264 000 tokens at block size 32, two of the heads: the finest blocks and the longest rows.
    add("call_264k_bs32", "call", 1, 2, 128, 33, 80, 100, 32, "bf16", "field", "static", 0.384, 0.5, 2, 0.15)
    # Guidance pair (B = 2) on an odd grid, block size 64, one mask per head by the paper's standardised thresholds.
    add("call_per_head_bs64", "call", 2, 12, 128, 17, 31, 45, 64, "bf16", "field", "zscore", 0.5, 0.5, 0, 0.285)
    # Head dimension 64 in bf16, 17 550 tokens, a mask that is kept over steps.
    add("attend_d64", "attend", 1, 12, 64, 13, 30, 45, 64, "bf16", "field", "random", 0.12, 0.5, 1, 0.32)
    # fp32 tensors at head dimension 128: the reference that a bf16 model is held against, and the search's read-out.
    add("attend_f32", "attend", 1, 8, 128, 8, 24, 32, 128, "f32", "field", "random", 0.2, 0.5, 1, 0.476)
    # Masks of 40 heads at 720p by the cumulative-mass rule.
    add("mask_per_head", "mask", 1, 40, 128, 21, 45, 80, 128, "bf16", "field", "dynamic", 0.9, 0.5, 0, 0.149)
    # Token-level order on 8192 tokens: one threshold of a sweep.
    add("tokens_8k", "tokens", 1, 2, 64, 8, 32, 32, 32, "f32", "field", "zscore", 0.5, 1.0, 2, 0.539)
    # The search's objective on its proxy task: token scores, links, attention matrices, norms.
    add("proxy_2k", "proxy", 1, 2, 64, 8, 16, 16, 32, "f32", "drift", "zscore", 0.0, 1.0, 2, 0.5)
    return out


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("call", "call", "call", "attend", "attend", "mask", "tokens", "proxy"))
    lam = rng.choice((0.3, 0.5, 0.7))
    for _ in range(1000):
        Nf = rng.randint(4, 33)
        Hg, Wg = _log_int(rng, 8, 80), _log_int(rng, 8, 100)
        N = Nf * Hg * Wg
        Bs = rng.choice((32, 64, 128, 128))
        if kind == "call":
            dtype, d = rng.choice((("bf16", 128), ("bf16", 128), ("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)))
            B, H = rng.choice((1, 1, 2)), _log_int(rng, 2, 40)
            most = 2.4e13 if (dtype, d) == ("bf16", 128) else 3.0e11 if d == 64 else 1.2e11
            mode = rng.choice(("static", "dynamic", "zscore", "uniform"))
            par = {"static": rng.uniform(0.04, 0.3), "dynamic": rng.uniform(0.7, 0.95), "zscore": rng.uniform(0.0, 1.0),
                   "uniform": rng.uniform(0.04, 0.3)}[mode]
            fuse = rng.choice((0, 1, 2))
            if 4.0 * d * N * N * B * H * 0.45 > most or N > 264000 or N < 256 or (fuse == 0 and B * H * (N / Bs) ** 2 > 6e7):
                continue
            return _case(kind, B, H, d, Nf, Hg, Wg, Bs, dtype, rng.choice(("field", "blob")), mode, round(par, 3), lam, fuse, 0.35)
        if kind == "attend":
            dtype, d = rng.choice((("bf16", 64), ("f32", 64), ("f32", 128), ("bf16", 128)))
            B, H = rng.choice((1, 1, 2)), _log_int(rng, 2, 16)
            par = round(rng.uniform(0.05, 0.4), 3)
            if 4.0 * d * N * N * B * H * 0.5 > (1.2e11 if d == 128 and dtype == "f32" else 3.0e11) or N < 256:
                continue
            return _case(kind, B, H, d, Nf, Hg, Wg, Bs, dtype, "field", "random", par, lam, rng.choice((0, 1)), 0.5)
        if kind == "mask":
            Sb = -(-N // Bs)
            B, H = 1, _log_int(rng, 2, 40)
            if N < 2048 or H * Sb * Sb > 1.5e7 or Sb > 2400:
                continue
            mode = rng.choice(("static", "dynamic", "zscore"))
            par = {"static": rng.uniform(0.04, 0.3), "dynamic": rng.uniform(0.7, 0.95), "zscore": rng.uniform(0.0, 1.0)}[mode]
            return _case(kind, B, H, 128, Nf, Hg, Wg, Bs, "bf16", "field", mode, round(par, 3), lam, 0, 0.35)
        if kind == "tokens":
            if N > 8192 or N < 1024 or Hg * Wg > 4096:
                continue
            return _case(kind, 1, 2, 64, Nf, Hg, Wg, rng.choice((32, 64)), "f32", "field", "zscore", round(rng.uniform(-1, 1), 3),
                         rng.choice((0.5, 1.0)), 2, 0.5)
        if N > 2048 or N < 512:
            continue
        return _case(kind, 1, rng.choice((1, 2)), 64, Nf, Hg, Wg, 32, "f32", "drift", "zscore", round(rng.uniform(-1, 1), 3),
                     1.0, 1, 0.5)
    raise RuntimeError("no case found")


# ---- inputs ------------------------------------------------------------------------------------------------

def _grid(case, device):
    Nt = case["Hg"] * case["Wg"]
    p = torch.arange(case["Nf"] * Nt, device=device)
    r = p % Nt
    return (p // Nt).float(), (r // case["Wg"]).float(), (r % case["Wg"]).float()


def _qkv(case, seed, device="cuda"):
    """Q, K, V [B, H, N, d] in the case's dtype."""
    B, H, d, Nf, Hg, Wg = (case[k] for k in ("B", "H", "d", "Nf", "Hg", "Wg"))
    N = Nf * Hg * Wg
    g = torch.Generator(device=device).manual_seed(seed * 7919 + 17)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    out = [torch.empty((B, H, N, d), dtype=dt, device=device) for _ in range(3)]
    t, y, x = _grid(case, device)

    def randn(*s):
        return torch.randn(*s, generator=g, device=device)

    for b in range(B):
        for h in range(H):
            if case["recipe"] == "iid":
                q, k = randn(N, d), randn(N, d)
            elif case["recipe"] == "drift":
                f = torch.empty(Nf, Hg * Wg, d, device=device)
                f[0] = randn(Hg * Wg, d)
                for i in range(1, Nf):
                    f[i] = math.sqrt(1 - 0.15 ** 2) * f[i - 1] + 0.15 * randn(Hg * Wg, d)
                q = k = f.view(N, d)
            else:
                freq, phi, blob = randn(3, d), torch.rand(d, generator=g, device=device), randn(d)
                f = math.sqrt(2.0) * torch.cos(2 * math.pi * (t[:, None] / Nf * freq[0] + y[:, None] / Hg * freq[1] +
                                                              x[:, None] / Wg * freq[2] + phi))
                if case["recipe"] == "blob":
                    cy, cx = 0.2 * Hg + 0.6 * Hg * t / max(1, Nf - 1), 0.15 * Wg + 0.7 * Wg * t / max(1, Nf - 1)
                    f += (1.5 * torch.exp(-((y - cy) ** 2 + (x - cx) ** 2) / (2 * (Hg / 6.0) ** 2)))[:, None] * blob
                q, k = f + 0.3 * randn(N, d), f + 0.3 * randn(N, d)
            out[0][b, h], out[1][b, h], out[2][b, h] = q.to(dt), k.to(dt), randn(N, d).to(dt)
    return out


def _block_scores(case, seed, device="cuda"):
    """Block scores [B, H, Sb, Sb] as a layer's pooled queries and keys give them: the field at the blocks' centres."""
    B, H, d, Bs = case["B"], case["H"], case["d"], case["Bs"]
    N = case["Nf"] * case["Hg"] * case["Wg"]
    Sb = -(-N // Bs)
    g = torch.Generator(device=device).manual_seed(seed * 104729 + 5)
    at = (torch.arange(Sb, device=device) * Bs + Bs // 2).clamp(max=N - 1)
    t, y, x = (v[at] for v in _grid(case, device))
    out = torch.empty((B, H, Sb, Sb), dtype=torch.float32, device=device)
    for b in range(B):
        for h in range(H):
            freq = torch.randn(3, d, generator=g, device=device)
            phi = torch.rand(d, generator=g, device=device)
            f = math.sqrt(2.0) * torch.cos(2 * math.pi * (t[:, None] / case["Nf"] * freq[0] + y[:, None] / case["Hg"] * freq[1] +
                                                          x[:, None] / case["Wg"] * freq[2] + phi))
            q = f + 0.05 * torch.randn(Sb, d, generator=g, device=device)
            out[b, h] = q @ f.T / math.sqrt(d)
    return out


def _random_mask(case, seed, device="cuda"):
    """CSR of block masks [B, masks]: every block of the query block's own and neighbouring frames, and a random share
    `par` of the others."""
    N, Nt, Bs = case["Nf"] * case["Hg"] * case["Wg"], case["Hg"] * case["Wg"], case["Bs"]
    Sb = -(-N // Bs)
    masks = case["H"] if case["fuse"] == 0 else 1
    g = torch.Generator(device=device).manual_seed(seed * 65537 + 3)
    first = torch.arange(Sb, device=device) * Bs // Nt
    last = ((torch.arange(Sb, device=device) + 1) * Bs).clamp(max=N).sub(1) // Nt
    gap = torch.maximum(first[None, :] - last[:, None], first[:, None] - last[None, :]).clamp(min=0)
    keep = (gap <= 1) | (torch.rand(case["B"], masks, Sb, Sb, generator=g, device=device) < case["par"])
    rowptr = torch.zeros(case["B"], masks, Sb + 1, dtype=torch.int32, device=device)
    rowptr[..., 1:] = keep.sum(-1).cumsum(-1)
    cap = int(rowptr[..., -1].max())
    colidx = torch.zeros(case["B"], masks, cap, dtype=torch.int32, device=device)
    for b in range(case["B"]):
        for m in range(masks):
            cols = keep[b, m].nonzero()[:, 1].int()
            colidx[b, m, :cols.numel()] = cols
    return keep, rowptr, colidx, cap


def _params(case):
    if case["kind"] in ("tokens", "proxy") or case["mode"] == "zscore":
        return dr.MaskParams(head_fuse=case["fuse"], tau_far=case["par"] + 0.3)
    return dr.MaskParams(head_fuse=case["fuse"])


def prepare(case, seed):
    kind, Bs, dev = case["kind"], case["Bs"], "cuda"
    geo = (case["Nf"], case["Hg"], case["Wg"], Bs)
    N = case["Nf"] * case["Hg"] * case["Wg"]
    Sb = -(-N // Bs)
    s = dict(case=case, ctx=dr.Context(0), params=_params(case))
    masks = case["H"] if case["fuse"] == 0 else 1
    if kind == "proxy":
        s["Q"], s["K"], _ = _qkv(case, seed)
        return s
    if kind == "attend":
        s["Q"], s["K"], s["V"] = _qkv(case, seed)
        s["shape"] = dr.shape_of(s["Q"], *geo)
        _, s["rowptr"], s["colidx"], s["cap"] = _random_mask(case, seed)
        s["masks"] = masks
        s["O"] = torch.empty_like(s["Q"])
        s["lse"] = torch.empty(s["Q"].shape[:3], dtype=torch.float32, device=dev)
        return s
    if kind == "call":
        s["Q"], s["K"], s["V"] = _qkv(case, seed)
        s["shape"] = dr.shape_of(s["Q"], *geo)
        s["O"] = torch.empty_like(s["Q"])
        s["scores"] = torch.empty((case["B"], masks, Sb, Sb), dtype=torch.float32, device=dev)
    elif kind == "mask":
        like = torch.empty((case["B"], case["H"], N, 1), dtype=torch.bfloat16, device=dev).expand(-1, -1, -1, case["d"])
        s["scores"] = _block_scores(case, seed)
        s["shape"] = dr.Shape(case["B"], case["H"], N, case["d"], *geo, 1, 0, like.shape[1] * N * case["d"], N * case["d"], case["d"])
    else:
        q, k, _ = _qkv(case, seed)
        s["shape"] = dr.shape_of(q, *geo)
        n_fused = case["fuse"] or 1
        s["scores"] = sum(q[:, h] @ k[:, h].transpose(-1, -2) for h in range(n_fused)).div_(n_fused * math.sqrt(case["d"]))[:, None].contiguous()
        s["links"] = torch.empty((case["B"], 1, N, N), dtype=torch.uint8, device=dev)
    s["masks"] = masks
    s["cap"], _ = dr.dr_mask_capacity(s["ctx"], s["shape"], case["lam"], s["params"])
    s["rowptr"] = torch.zeros((case["B"], masks, Sb + 1), dtype=torch.int32, device=dev)
    s["colidx"] = torch.zeros((case["B"], masks, s["cap"]), dtype=torch.int32, device=dev)
    s["nnz"] = torch.zeros((case["B"], masks), dtype=torch.int64, device=dev)
    return s


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "proxy":
        loss, nmse, sparsity = proxy_eval.proxy_loss(s["ctx"], s["Q"], s["K"], c["Nf"], c["Hg"], c["Wg"], c["Bs"],
                                                     proxy_eval.MODE_TOKENS, c["par"], c["lam"], s["params"])
        return {"loss": loss, "nmse": nmse, "sparsity": sparsity}
    if kind == "tokens":
        dr.dr_build_mask_tokens(s["ctx"], s["shape"], c["par"], c["lam"], s["params"], s["scores"], s["rowptr"], s["colidx"],
                                s["cap"], s["nnz"], s["links"])
        return {"rowptr": s["rowptr"], "colidx": s["colidx"], "nnz": s["nnz"], "links": s["links"]}
    if kind == "attend":
        dr.dr_sparse_attn_fwd(s["ctx"], s["shape"], s["Q"], s["K"], s["V"], s["rowptr"], s["colidx"], s["masks"], s["cap"],
                              s["O"], s["lse"])
        return {"O": s["O"], "lse": s["lse"]}
    if kind == "call":
        dr.dr_block_scores(s["ctx"], s["shape"], s["Q"], s["K"], c["fuse"], s["scores"])
    dr.dr_build_mask(s["ctx"], s["shape"], MODES[c["mode"]], c["par"], c["lam"], s["params"], s["scores"], s["rowptr"],
                     s["colidx"], s["cap"], s["nnz"])
    if kind == "mask":
        return {"rowptr": s["rowptr"], "colidx": s["colidx"], "nnz": s["nnz"]}
    dr.dr_sparse_attn_fwd(s["ctx"], s["shape"], s["Q"], s["K"], s["V"], s["rowptr"], s["colidx"], s["masks"], s["cap"], s["O"])
    return {"scores": s["scores"], "O": s["O"]}


def work(case):
    """Inputs once, outputs once; two products over the kept block pairs."""
    B, H, d, Bs = case["B"], case["H"], case["d"], case["Bs"]
    N = case["Nf"] * case["Hg"] * case["Wg"]
    Sb = -(-N // Bs)
    es = 2 if case["dtype"] == "bf16" else 4
    masks = case["H"] if case["fuse"] == 0 else 1
    csr = 4.0 * B * masks * Sb * Sb * case["kept"]
    kind = case["kind"]
    if kind == "mask":
        return {"bytes": 4.0 * B * masks * Sb * Sb + csr, "flops": 4.0 * B * masks * Sb * Sb}
    if kind == "tokens":      # scores in, link bytes out; mean, deviation and test of every token pair
        return {"bytes": 5.0 * B * N * N, "flops": 6.0 * B * N * N}
    if kind == "proxy":       # features in; the dense and the kept attention matrix, and the token scores
        return {"bytes": 2.0 * B * H * N * d * es, "flops": 2.0 * d * B * H * N * N * (2.0 + case["kept"])}
    flops = 4.0 * d * B * H * float(N) * N * case["kept"]
    moved = 4.0 * B * H * N * d * es
    if kind == "attend":
        return {"bytes": moved + csr + 4.0 * B * H * N, "flops": flops}
    scored = case["fuse"] or H
    return {"bytes": moved + csr + 4.0 * B * masks * Sb * Sb, "flops": flops + 2.0 * d * B * scored * float(Sb) * Sb}


def tolerance(case):
    if case["kind"] in ("mask", "tokens"):
        return "exact"
    if case["kind"] == "proxy":      # a token score on the threshold can decide one block of the mask: 1 / Sb^2 of the sparsity
        return {"rel": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ---- the same in 64 bits ---------------------------------------------------------------------------------

def _exact_scores(case, Q, K):
    B, H, N, d = Q.shape
    Bs, heads = case["Bs"], case["fuse"] or case["H"]
    Sb = -(-N // Bs)
    n = torch.full((Sb,), Bs, dtype=torch.float64, device=Q.device)
    n[-1] = N - (Sb - 1) * Bs

    def pool(x):
        y = torch.zeros(Sb * Bs, d, dtype=torch.float64, device=x.device)
        y[:N] = x.double()
        return y.view(Sb, Bs, d).sum(1) / n[:, None]

    out = torch.zeros(B, 1 if case["fuse"] else H, Sb, Sb, dtype=torch.float64, device=Q.device)
    for b in range(B):
        for h in range(heads):
            s = pool(Q[b, h]) @ pool(K[b, h]).T / math.sqrt(d)
            if case["fuse"]:
                out[b, 0] += s / heads
            else:
                out[b, h] = s
    return out


def _exact_attention(case, Q, K, V, keep):
    B, H, N, d = Q.shape
    Bs, Sb = case["Bs"], keep.shape[-1]
    O = torch.zeros(B, H, N, d, dtype=torch.float64, device=Q.device)
    lse = torch.empty(B, H, N, dtype=torch.float64, device=Q.device)
    step = max(1, 4096 // Bs)
    for b in range(B):
        for h in range(H):
            kk = keep[b, h if keep.shape[1] > 1 else 0]
            Kd, Vd = K[b, h].double(), V[b, h].double()
            for q0 in range(0, Sb, step):
                rows = slice(q0 * Bs, min(N, (q0 + step) * Bs))
                allowed = kk[q0:q0 + step].repeat_interleave(Bs, 0)[:rows.stop - rows.start].repeat_interleave(Bs, 1)[:, :N]
                s = (Q[b, h, rows].double() @ Kd.T / math.sqrt(d)).masked_fill(~allowed, -math.inf)
                lse[b, h, rows] = torch.logsumexp(s, 1)
                O[b, h, rows] = torch.softmax(s, 1) @ Vd
    return {"O": O, "lse": lse}


def exact(case, seed):
    if case["kind"] in ("mask", "tokens", "proxy"):
        return None
    Q, K, V = _qkv(case, seed)
    if case["kind"] == "attend":
        return _exact_attention(case, Q, K, V, _random_mask(case, seed)[0])
    return {"scores": _exact_scores(case, Q, K), "O": None}
