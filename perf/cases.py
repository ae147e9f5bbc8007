"""Workloads of the cache-hit attention path, for timing and for comparing outputs.

A case is one call, or the few calls a serving program makes back to back, of
the public binding on inputs of a size that the video backbones named in the
synthetic workloads (or their smaller and odd-sized relatives) produce.
Inputs are smooth spatiotemporal fields plus noise on the latent grid, as in
the benchmark: attention that is local in space and time, block masks that
keep 10-50 % of the pairs, and target rows from a box on the grid.

Kinds (``case["kind"]``):

  request    build_block_mask, merge_target_rows, block_sparse_attn with the
             LSE: a whole layer of a request without preallocated buffers
  record     MaskBank.record: a historical layer's connectivity stored
             bit-packed
  build      build_block_mask and merge_target_rows with dense text columns
             (the uint8 form)
  reuse      MaskBank.lists for a target, then block_sparse_attn_lists: one
             layer of a cache-hit request
  attention  block_sparse_attn from a uint8 mask on [B, N, H, d] storage
  region     the middle-layer variant: lists restricted to active rows and
             context keys, attention of the active rows
  regions    region_weights, region_block_flags and latent_fusion: set up
             per request and blended per step
  exact      block_mass_exact and select_block_mask: the builder on
             token-level mass
  signature  signature_sim: ranking a bank of early signatures
"""
import math

import torch

import paper_2609_32420_amd as P

DEV = "cuda"
SIGMA_HIST = 0.2   # std of the historical copy's perturbation
NOISE = 0.5        # std of the noise on Q, K and V
ALPHA = 1.85       # amplitude of the smooth fields
TIE = 1e-6         # width of the builder's tie rule
PATCH = (1, 2, 2)  # latent elements per token
RADII = (2, 3)     # active and context dilation


def listed():
    return [
        # the smallest request the repository's smoke test runs: launches and host time
        _attn("request_tiny", "request", 1, 2, (3, 8, 8), 0, 64, 64, 0.9),
        # a short odd-sized clip, two guidance branches, 64-token blocks with a ragged tail
        _attn("request_2k", "request", 2, 6, (7, 13, 21), 77, 128, 64, 0.9),
        # recording a Wan2.1-1.3B layer (32K tokens) into the bank
        _attn("record_32k", "record", 1, 12, (21, 30, 52), 0, 128, 128, 0.9),
        # recording a Wan2.1-14B layer (75.6K tokens, 40 heads)
        _attn("record_75k", "record", 1, 40, (21, 45, 80), 0, 128, 128, 0.9),
        # CogVideoX-5B layer (text and video tokens, 64 channels), uint8 masks
        _attn("build_17k", "build", 1, 48, (13, 30, 45), 226, 64, 128, 0.85),
        # a cache-hit layer at 32K tokens, the benchmark's headline shape
        _attn("reuse_32k", "reuse", 1, 12, (21, 30, 52), 0, 128, 128, 0.9),
        # attention with the LSE at d = 64 on the projection's own [B, N, H, d] layout
        _attn("attention_17k", "attention", 1, 48, (13, 30, 45), 226, 64, 128, 0.85),
        # the longest layer: HunyuanVideo, 119K tokens
        _attn("reuse_119k", "reuse", 1, 24, (33, 45, 80), 256, 128, 128, 0.8),
        # a middle layer restricted to the active region at 32K tokens
        _attn("region_32k", "region", 1, 12, (21, 30, 52), 0, 128, 128, 0.9),
        # regions, block flags and one latent blend at the 32K grid
        {"name": "regions_32k", "kind": "regions", "batch": 1, "grid_t": 21, "grid_h": 30, "grid_w": 52,
         "channels": 16, "text": 0, "block": 128},
        # the token-level builder at 32K tokens
        _attn("exact_32k", "exact", 1, 12, (21, 30, 52), 0, 128, 128, 0.9),
        # two early signatures ranked against the bank of 4096
        {"name": "signature_4k", "kind": "signature", "queries": 2, "rows": 4096, "dim": 3072, "topk": 8},
    ]


def _attn(name, kind, batch, heads, grid, text, d, block, tau):
    c = {"kind": kind, "batch": batch, "heads": heads, "grid_t": grid[0], "grid_h": grid[1], "grid_w": grid[2],
         "text": text, "d": d, "block": block, "tau": tau}
    return dict(c, name=name) if name else c


def draw(rng):
    kind = rng.choice(["request", "record", "build", "reuse", "attention", "region", "regions", "exact", "signature"])
    if kind == "signature":
        return {"kind": kind, "queries": rng.randint(1, 9), "rows": int(_log(rng, 200, 20000)),
                "dim": 4 * int(_log(rng, 32, 1024)), "topk": rng.choice([1, 4, 8, 16, 50])}
    most = {"request": 5000, "exact": 40000}.get(kind, 120000)
    n = _log(rng, 200, most)
    t = rng.randint(3, 33)
    t = min(t, max(1, int(n / 25)))
    h = max(4, int(math.sqrt(n / t * rng.uniform(0.4, 1.0))))
    w = max(4, int(n / t / h))
    if kind == "regions":
        return {"kind": kind, "batch": rng.randint(1, 2), "grid_t": t, "grid_h": h, "grid_w": w,
                "channels": rng.choice([4, 16, 24, 48]), "text": rng.choice([0, 0, 77, 226]),
                "block": rng.choice([64, 128])}
    text = rng.choice([0, 0, 77, 226, 256])
    n = text + t * h * w
    d = rng.choice([64, 128, 128])
    block = 128 if n > 64 * 1500 else rng.choice([64, 128, 128])
    batch = rng.choice([1, 1, 2])
    # heads of a backbone, as far as the work stays below the largest listed case's
    cost = {"exact": 2.0 * d * n * n, "record": 0.0, "build": 0.0}.get(kind, 1.6 * d * n * n)
    nb = -(-n // block)
    fit = min(8e12 / max(cost * batch, 1.0), 1.5e7 / (batch * nb * nb), 1.5e9 / (batch * n * d * 2))
    heads = max(1, min(rng.choice([2, 6, 12, 24, 40, 48]), int(fit)))
    return _attn("", kind, batch, heads, (t, h, w), text, d, block, rng.choice([0.8, 0.85, 0.9]))


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


# ---------------------------------------------------------------- inputs

def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _tokens(c):
    return c["text"] + c["grid_t"] * c["grid_h"] * c["grid_w"]


def _blocks(c):
    return -(-_tokens(c) // c["block"])


def _basis(c):
    """cos and sin of 2 pi <f, (t/T, y/H, x/W)> over the tokens, f in {0,1,2}^3 but the origin."""
    axes = [torch.arange(m, device=DEV, dtype=torch.float32) / m for m in (c["grid_t"], c["grid_h"], c["grid_w"])]
    pos = torch.stack(torch.meshgrid(*axes, indexing="ij"), -1).reshape(-1, 3)
    f = torch.tensor([(a, b, e) for a in range(3) for b in range(3) for e in range(3)][1:], device=DEV,
                     dtype=torch.float32)
    ph = 2.0 * math.pi * (pos[:, None, :] * f[None, :, :]).sum(-1)
    return torch.cat([ph.cos(), ph.sin()], 1)


def _coefficients(g, channels):
    """Four sinusoids per channel with N(0, 1/4) amplitudes and uniform phases, on the basis."""
    pick = torch.randint(0, 26, (channels, 4), generator=g, device=DEV)
    amp = ALPHA * 0.5 * torch.randn(channels, 4, generator=g, device=DEV)
    phi = 2.0 * math.pi * torch.rand(channels, 4, generator=g, device=DEV)
    out = torch.zeros(channels, 52, device=DEV)
    out.scatter_add_(1, pick, amp * phi.sin())
    out.scatter_add_(1, pick + 26, amp * phi.cos())
    return out


def _qkv(c, seed, names):
    """The tensors of ``names`` (q, k, v, q_hist, k_hist) as bf16 [B, H, N, d]."""
    g = _gen(seed, 1)
    B, H, N, d, nt = c["batch"], c["heads"], _tokens(c), c["d"], c["text"]
    basis = _basis(c)
    cq = _coefficients(g, H * d).view(H, d, 52)
    cv = _coefficients(g, H * d).view(H, d, 52)
    out = {n: torch.empty(B, H, N, d, dtype=torch.bfloat16, device=DEV) for n in names}
    for b in range(B):
        for h in range(H):
            fields = {}
            for name, co in (("q", cq), ("k", cq), ("v", cv)):
                if name not in names and name + "_hist" not in names:
                    continue
                x = torch.randn(N, d, generator=g, device=DEV)
                x[nt:].mul_(NOISE)
                if name not in fields:
                    x[nt:] += _field(basis, co[h])
                x = x.to(torch.bfloat16)
                if name in names:
                    out[name][b, h] = x
                if name + "_hist" in names:
                    out[name + "_hist"][b, h] = x + SIGMA_HIST * torch.randn(N, d, generator=g, device=DEV)
    return out


def _field(basis, co):
    # accumulated by the frequencies, not by a library product, so that it is the same everywhere
    out = torch.zeros(basis.shape[0], co.shape[0], device=DEV)
    for m in range(basis.shape[1]):
        out.addcmul_(basis[:, m:m + 1], co[:, m].unsqueeze(0))
    return out


def _target_flags(c, seed):
    """(rows, cols or None) uint8 [B, nB]: blocks touched by a box on the grid, and the text blocks."""
    g = torch.Generator().manual_seed(int(seed) * 1000003 + 2)
    B, nb, nt = c["batch"], _blocks(c), c["text"]
    T, H, W = c["grid_t"], c["grid_h"], c["grid_w"]
    tok = torch.zeros(B, _tokens(c), dtype=torch.bool)
    for b in range(B):
        u = torch.rand(3, generator=g).tolist()
        pt, ph, pw = max(1, T // 2), max(1, H // 10), max(1, W // 4)
        t, y, x = int(u[0] * (T - pt + 1)), int(u[1] * (H - ph + 1)), int(u[2] * (W - pw + 1))
        tok[b, nt:].view(T, H, W)[t:t + pt, y:y + ph, x:x + pw] = True
    tok[:, :nt] = True
    rows = _any_per_block(tok, nb, c["block"]).to(torch.uint8).to(DEV)
    if not nt:
        return rows, None
    text = torch.zeros(B, _tokens(c), dtype=torch.bool)
    text[:, :nt] = True
    return rows, _any_per_block(text, nb, c["block"]).to(torch.uint8).to(DEV)


def _any_per_block(tok, nb, bs):
    pad = torch.zeros(tok.shape[0], nb * bs, dtype=torch.bool, device=tok.device)
    pad[:, :tok.shape[1]] = tok
    return pad.view(tok.shape[0], nb, bs).any(-1)


def _evidence(c, seed):
    """An ellipse per frame that drifts over the frames, a quarter of the frames empty: uint8 [B, T, H, W]."""
    g = torch.Generator().manual_seed(int(seed) * 1000003 + 3)
    B, T, H, W = c["batch"], c["grid_t"], c["grid_h"], c["grid_w"]
    yy, xx = torch.meshgrid(torch.arange(H), torch.arange(W), indexing="ij")
    out = torch.zeros(B, T, H, W, dtype=torch.uint8)
    for b in range(B):
        u = torch.rand(6, generator=g).tolist()
        empty = torch.rand(T, generator=g) < 0.25
        empty[int(u[4] * T)] = False
        for t in range(T):
            cy = (0.3 + 0.4 * u[0] + 0.2 * (u[2] - 0.5) * t / T) * H
            cx = (0.3 + 0.4 * u[1] + 0.2 * (u[3] - 0.5) * t / T) * W
            r = ((yy - cy) / (H / 5.0)) ** 2 + ((xx - cx) / (W / 5.0)) ** 2
            if not empty[t]:
                out[b, t] = (r <= 1.0).to(torch.uint8)
    return out.to(DEV)


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device=DEV)


def _lists_out(c):
    R = c["batch"] * c["heads"] * _blocks(c)
    return (torch.zeros(R + 1, dtype=torch.int32, device=DEV),
            torch.zeros(R * _blocks(c), dtype=torch.int32, device=DEV),
            torch.zeros(R, dtype=torch.int32, device=DEV))


# ---------------------------------------------------------------- the cases

def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind == "signature":
        g = _gen(seed, 4)
        bank = torch.randn(c["rows"], c["dim"], generator=g, device=DEV)
        query = torch.randn(c["queries"], c["dim"], generator=g, device=DEV)
        # half of the queries are near-duplicates of a stored request
        for i in range(1, c["queries"], 2):
            query[i] = bank[(i * 7919 + int(seed)) % c["rows"]] + 0.5 * query[i]
        return {"case": c, "query": query, "bank": bank, "topk": min(c["topk"], c["rows"]),
                "workspace": P.signature_sim_workspace(c["queries"], c["rows"], min(c["topk"], c["rows"]), DEV)}
    if kind == "regions":
        g = _gen(seed, 5)
        shape = (c["batch"], c["channels"], c["grid_t"] * PATCH[0], c["grid_h"] * PATCH[1], c["grid_w"] * PATCH[2])
        grid = (c["batch"], c["grid_t"], c["grid_h"], c["grid_w"])
        return {"case": c, "evidence": _evidence(c, seed), "z_target": torch.randn(shape, generator=g, device=DEV),
                "z_hist": torch.randn(shape, generator=g, device=DEV),
                "region": (torch.empty(grid, dtype=torch.uint8, device=DEV), torch.empty(grid, device=DEV)),
                "blend": torch.empty(shape, device=DEV)}
    names = {"request": ("q", "k", "v", "q_hist", "k_hist"), "record": ("q_hist", "k_hist"),
             "build": ("q_hist", "k_hist"), "exact": ("q_hist", "k_hist")}.get(kind, ("q", "k", "v"))
    x = _qkv(c, seed, names)
    B, H, nb, N, d, bs = c["batch"], c["heads"], _blocks(c), _tokens(c), c["d"], c["block"]
    st = dict(x, case=c)
    if kind in ("request", "build", "reuse"):
        st["rows"], st["cols"] = _target_flags(c, seed)
    if kind == "record":
        st["bank"] = P.MaskBank(1, 1, 1, B, H, nb, device=DEV)
        st["workspace"] = P.build_block_mask_workspace(x["q_hist"], bs)
    elif kind == "build":
        st["out"] = torch.empty(B, H, nb, nb, dtype=torch.uint8, device=DEV)
        st["workspace"] = P.build_block_mask_workspace(x["q_hist"], bs)
    elif kind == "exact":
        st["mass"] = torch.empty(B, H, nb, nb, dtype=torch.float64, device=DEV)
        st["workspace"] = None
    elif kind == "attention":
        for n in ("q", "k", "v"):
            st[n] = x[n].transpose(1, 2).contiguous().transpose(1, 2)
        st["mask"] = _widened(c, seed, _pooled_mask(c, x["q"], x["k"]))
        st["workspace"] = P.block_sparse_attn_workspace(st["q"], bs)
    elif kind in ("reuse", "region"):
        bank = P.MaskBank(1, 1, 1, B, H, nb, device=DEV)
        bank.bits[0, 0, 0] = _pack(_pooled_mask(c, x["q"], x["k"]))
        st["bank"] = bank
        st["lists"] = _lists_out(c)
        st["workspace"] = P.compact_block_mask_bits_workspace(bank.slot(0, 0, 0))
        st["out"] = torch.zeros(B, H, N, d, dtype=torch.bfloat16, device=DEV)
    if kind == "region":
        st["lists"] += (torch.zeros(1, dtype=torch.int32, device=DEV),)
        st["active"], st["context"] = _block_flags(c, seed)
    return st


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "signature":
        return P.signature_sim(state["query"], state["bank"], state["topk"], workspace=state["workspace"])
    if kind == "regions":
        region, weight = P.region_weights(state["evidence"], *RADII, out=state["region"])
        active, context = P.region_block_flags(region, c["text"], c["block"])
        z = P.latent_fusion(state["z_target"], state["z_hist"], weight, out=state["blend"])
        return region, weight, active, context, z
    bs, tau = c["block"], c["tau"]
    if kind == "request":
        mask = P.build_block_mask(state["q_hist"], state["k_hist"], bs, tau)
        P.merge_target_rows(mask, state["rows"], state["cols"])
        out, lse = P.block_sparse_attn(state["q"], state["k"], state["v"], mask, bs, return_lse=True)
        return mask, out, lse
    if kind == "record":
        return state["bank"].record(0, 0, 0, state["q_hist"], state["k_hist"], bs, tau, workspace=state["workspace"])
    if kind == "build":
        mask = P.build_block_mask(state["q_hist"], state["k_hist"], bs, tau, out=state["out"],
                                  workspace=state["workspace"])
        return P.merge_target_rows(mask, state["rows"], state["cols"])
    if kind == "exact":
        mass = P.block_mass_exact(state["q_hist"], state["k_hist"], bs, out=state["mass"])
        return mass, P.select_block_mask(mass, tau)
    if kind == "attention":
        return P.block_sparse_attn(state["q"], state["k"], state["v"], state["mask"], bs, return_lse=True,
                                   workspace=state["workspace"])
    attn = (_tokens(c), c["d"], bs)
    if kind == "reuse":
        lists = state["bank"].lists(0, 0, 0, state["rows"], state["cols"], trim=False, out=state["lists"],
                                    workspace=state["workspace"], attn=attn)
        return P.block_sparse_attn_lists(state["q"], state["k"], state["v"], lists, bs, out=state["out"])
    lists = P.compact_block_mask_bits_region(state["bank"].slot(0, 0, 0), state["active"], state["context"],
                                             out=state["lists"], workspace=state["workspace"], attn=attn)
    return P.block_sparse_attn_lists(state["q"], state["k"], state["v"], lists[:3], bs, out=state["out"],
                                     n_rows=lists[3])


def work(case):
    c = case
    kind = c["kind"]
    if kind == "signature":
        n = 4.0 * c["rows"] * c["dim"] + 4.0 * c["queries"] * c["dim"] + 8.0 * c["queries"] * c["topk"]
        return {"bytes": n, "flops": 2.0 * (c["queries"] + 1) * c["rows"] * c["dim"]}
    if kind == "regions":
        tok = float(c["batch"] * c["grid_t"] * c["grid_h"] * c["grid_w"])
        z = tok * PATCH[0] * PATCH[1] * PATCH[2] * c["channels"]
        return {"bytes": 12.0 * z + 6.0 * tok, "flops": 3.0 * z}
    N, d, BH, nb = float(_tokens(c)), c["d"], c["batch"] * c["heads"], _blocks(c)
    tensor = 2.0 * BH * N * d
    pairs = float(BH) * nb * nb
    score = 2.0 * BH * nb * nb * d
    if kind in ("record", "build"):
        return {"bytes": 2 * tensor + (pairs / 8 if kind == "record" else pairs), "flops": score}
    if kind == "exact":
        return {"bytes": 2 * tensor + 9.0 * pairs, "flops": 2.0 * BH * d * N * N}
    # the kept share of the block pairs, as counted on these inputs at the listed sizes
    kept = {"region": 0.05, "reuse": 0.12 if N > 1e5 else 0.23, "attention": 0.4}.get(kind, 0.5)
    flops = 4.0 * BH * d * N * N * kept
    if kind == "request":
        return {"bytes": 6 * tensor + pairs + 4.0 * BH * N, "flops": flops + score}
    return {"bytes": 4 * tensor + (pairs if kind == "attention" else pairs / 8), "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("record", "build"):
        return "exact"  # fp64 decisions, whole values
    if kind == "regions":
        return {"rel": 4e-7, "max": 1e-6, "differ": 0.0}  # fp32 arithmetic on whole distances
    if kind == "signature":
        return {"rel": 4e-7, "max": 1e-6, "differ": 0.0}  # fp64 sums rounded once to fp32
    if kind == "exact":
        # fp32 scores and sums of exponentials; a mask entry whose cut lies within that may differ
        return {"rel": 2e-6, "max": 2e-5, "differ": 1e-5}
    return {"rel": 8e-3, "max": 1e-1, "differ": 0.0}  # bf16 probabilities and outputs


# ---------------------------------------------------------------- in 64 bits

def exact(case, seed):
    c = case
    kind = c["kind"]
    st = prepare(c, seed)
    if kind == "signature":
        q, b = st["query"].double(), st["bank"].double()
        den = q.norm(dim=1)[:, None] * b.norm(dim=1)[None, :]
        cos = torch.where(den > 0, (q @ b.t()) / den, torch.zeros_like(den))
        sim, idx = cos.sort(dim=1, descending=True, stable=True)
        return idx[:, :st["topk"]].to(torch.int32), sim[:, :st["topk"]]
    if kind == "regions":
        region, weight = _region_weights(st["evidence"])
        active, context = _flags_of(c, region)
        w = weight.repeat_interleave(PATCH[0], 1).repeat_interleave(PATCH[1], 2).repeat_interleave(PATCH[2], 3)
        w = w.unsqueeze(1)
        z = w * st["z_target"].double() + (1.0 - w) * st["z_hist"].double()
        return region, weight, active, context, z
    if kind == "record":
        return _pack(_pooled_mask(c, st["q_hist"], st["k_hist"]))
    if kind == "build":
        return _widened(c, seed, _pooled_mask(c, st["q_hist"], st["k_hist"]))
    if kind == "exact":
        mass = _block_mass(c, st["q_hist"], st["k_hist"])
        return mass, _select(mass, mass, c["tau"])
    if kind == "request":
        mask = _widened(c, seed, _pooled_mask(c, st["q_hist"], st["k_hist"]))
        return (mask,) + _attention(c, st, mask, None)
    if kind == "attention":
        return _attention(c, st, st["mask"], None)
    mask = _unpack(st["bank"].slot(0, 0, 0), _blocks(c))
    if kind == "reuse":
        return _attention(c, st, _widened(c, seed, mask), None)[0]
    mask = mask & st["context"][:, None, None, :]
    return _attention(c, st, mask, st["active"])[0]


def _block_mean(c, x):
    """fp64 means over the valid tokens of each block, [B, H, nB, d]."""
    nb, bs, N = _blocks(c), c["block"], _tokens(c)
    out = torch.empty(x.shape[0], x.shape[1], nb, x.shape[3], dtype=torch.float64, device=x.device)
    for b in range(x.shape[0]):
        for h in range(x.shape[1]):
            t = torch.zeros(nb * bs, x.shape[3], dtype=torch.float64, device=x.device)
            t[:N] = x[b, h].double()
            out[b, h] = t.view(nb, bs, -1).sum(1)
    n = torch.full((nb, 1), float(bs), dtype=torch.float64, device=x.device)
    n[-1] = N - (nb - 1) * bs
    return out / n


def _pooled_mask(c, q, k):
    """The block mask of pooled scores, uint8 [B, H, nB, nB]."""
    qm, km = _block_mean(c, q), _block_mean(c, k)
    s = torch.stack([torch.stack([qm[b, h] @ km[b, h].t() for h in range(q.shape[1])]) for b in range(q.shape[0])])
    s = s / math.sqrt(c["d"])
    return _select(s, torch.softmax(s, -1), c["tau"])


def _select(score, mass, tau):
    """Smallest prefix by descending score whose share of the mass reaches tau; near ties to the lower index."""
    out = torch.empty(score.shape, dtype=torch.uint8, device=score.device)
    for b in range(score.shape[0]):
        for h in range(score.shape[1]):
            s, m = score[b, h], mass[b, h]
            v, order = s.sort(dim=-1, descending=True, stable=True)
            cum = m.gather(-1, order).cumsum(-1)
            k = ((cum < tau * m.sum(-1, keepdim=True)).sum(-1, keepdim=True) + 1).clamp(max=s.shape[-1])
            cut = v.gather(-1, k - 1)
            above = s > cut + TIE
            tied = (s - cut).abs() <= TIE
            out[b, h] = above | (tied & (tied.cumsum(-1) <= k - above.sum(-1, keepdim=True)))
    return out


def _widened(c, seed, mask):
    rows, cols = _target_flags(c, seed)
    mask = mask | rows[:, None, :, None]
    return mask if cols is None else mask | cols[:, None, None, :]


def _pack(mask):
    nb = mask.shape[-1]
    w = -(-nb // 64)
    pad = torch.zeros(*mask.shape[:-1], w * 64, dtype=torch.uint8, device=mask.device)
    pad[..., :nb] = mask
    shift = torch.arange(64, device=mask.device)
    return (pad.view(*mask.shape[:-1], w, 64).long() << shift).sum(-1)


def _unpack(bits, nb):
    shift = torch.arange(64, device=bits.device)
    return ((bits.unsqueeze(-1) >> shift) & 1).flatten(-2)[..., :nb].to(torch.uint8)


def _attention(c, st, mask, active):
    """(O, LSE) in fp64 over the kept blocks; rows of inactive query blocks stay zero."""
    N, d, bs = _tokens(c), c["d"], c["block"]
    out = torch.zeros(c["batch"], c["heads"], N, d, dtype=torch.float64, device=DEV)
    lse = torch.zeros(c["batch"], c["heads"], N, dtype=torch.float64, device=DEV)
    kept = mask.cpu()
    act = None if active is None else active.cpu()
    step = torch.arange(bs, device=DEV)
    for b in range(c["batch"]):
        for h in range(c["heads"]):
            q, k, v = (st[n][b, h].double() for n in ("q", "k", "v"))
            q = q / math.sqrt(d)
            for i in range(_blocks(c)):
                if act is not None and not act[b, i]:
                    continue
                blocks = kept[b, h, i].nonzero().flatten().to(DEV)
                tok = (blocks[:, None] * bs + step[None, :]).flatten()
                tok = tok[tok < N]
                s = q[i * bs:(i + 1) * bs] @ k[tok].t()
                m = torch.logsumexp(s, -1, keepdim=True)
                out[b, h, i * bs:(i + 1) * bs] = (s - m).exp() @ v[tok]
                lse[b, h, i * bs:(i + 1) * bs] = m[:, 0]
    return out, lse


def _block_mass(c, q_hist, k_hist):
    N, nb, bs = _tokens(c), _blocks(c), c["block"]
    out = torch.zeros(c["batch"], c["heads"], nb, nb, dtype=torch.float64, device=DEV)
    for b in range(c["batch"]):
        for h in range(c["heads"]):
            q, k = q_hist[b, h].double() / math.sqrt(c["d"]), k_hist[b, h].double()
            for i0 in range(0, nb, 16):
                p = torch.softmax(q[i0 * bs:(i0 + 16) * bs] @ k.t(), -1)
                pad = torch.zeros(p.shape[0], nb * bs, dtype=torch.float64, device=DEV)
                pad[:, :N] = p
                per = pad.view(-1, nb, bs).sum(-1)
                for i in range(i0, min(i0 + 16, nb)):
                    out[b, h, i] = per[(i - i0) * bs:(i - i0 + 1) * bs].mean(0)
    return out


def _region_weights(evidence):
    """(codes, W) from the capped Chebyshev distance, by repeated 3 x 3 dilation."""
    ra, reach = RADII[0], sum(RADII)
    cur = (evidence != 0).float()
    dist = torch.where(cur > 0, 0, reach + 1)
    for r in range(1, reach + 1):
        cur = torch.nn.functional.max_pool2d(cur, 3, 1, 1)
        dist = torch.where((cur > 0) & (dist > r), r, dist)
    region = ((dist <= 0).to(torch.uint8) + (dist <= ra).to(torch.uint8) + (dist <= reach).to(torch.uint8))
    band = region == 2
    far = torch.where(band, dist, 1).amax(dim=(1, 2, 3), keepdim=True)
    s = dist.double() / far.double()
    w = torch.where(band, 1.0 - s * s * (3.0 - 2.0 * s), (region == 3).double())
    return region, w


def _flags_of(c, region):
    B, nt = c["batch"], c["text"]
    code = torch.full((B, _tokens(c)), 3, dtype=torch.uint8, device=region.device)
    code[:, nt:] = region.reshape(B, -1)
    nb, bs = _blocks(c), c["block"]
    return (_any_per_block(code >= 2, nb, bs).to(torch.uint8), _any_per_block(code >= 1, nb, bs).to(torch.uint8))


def _block_flags(c, seed):
    return _flags_of(c, _region_weights(_evidence(c, seed))[0])
