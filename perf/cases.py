"""Performance cases of the token-scoring path: what a user's program calls, over
the range of shapes, storage types and options it is used with.

A case is a dict of plain values.  `entry` names the public call:

  prune        a Pruner kept by the program, called on packed Q and K
  views        prune_views on per-layer views of a key/value cache
  ragged       a RaggedPruner kept by the program (images of different sizes)
  progressive  three StagePruner operations on three source layers, the next
               operation's candidate keys and, at the end, the kept tokens' hidden
               states gathered with compact_tokens

`value_std` is the element deviation of Q and K: 0 selects 1/sqrt(d) (logits within
a few thousandths of their mean, the repository's benchmark recipe); 1 gives logits
of unit spread, as the attention of a trained model has.  About 5 % of an image's
tokens, in clusters, have their keys shifted toward the mean query.
"""
import math
import random

import torch

import paper_2608_23253_amd as E

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(name, entry, **kw):
    c = dict(name=name, entry=entry, batch=1, layers=4, heads=32, kv_heads=32, head_dim=128,
             text=64, grid_h=24, grid_w=24, keep=128, cells=4, lam=0.1, mode="mean_logit",
             dtype="bf16", value_std=0.0, sizes_seed=0)
    c.update(kw)
    return c


def listed():
    qwen = dict(batch=32, heads=28, kv_heads=4, text=96, grid_h=32, grid_w=32, keep=256)
    hires = dict(batch=16, layers=6, text=128, grid_h=64, grid_w=64, keep=512)
    return [
        # the smallest call: launches and host time only
        _case("tiny_f32", "prune", layers=2, heads=4, kv_heads=4, head_dim=64, text=16, grid_h=8,
              grid_w=8, keep=16, lam=0.5, dtype="f32"),
        # one interactive request: a LLaVA-1.5-7B image read in place from the model's
        # caches, where latency counts
        _case("llava_single_views", "views"),
        # the serving batch of the benchmark: LLaVA-1.5-7B, 64 images, both readings
        _case("llava_batch", "prune", batch=64),
        _case("llava_batch_prob", "prune", batch=64, mode="mean_prob"),
        # grouped-query attention: Qwen2-VL-7B, 32 images, both readings
        _case("qwen2vl_batch", "prune", **qwen),
        _case("qwen2vl_batch_prob", "prune", mode="mean_prob", **qwen),
        # half-precision checkpoints, with the logit spread of a trained model
        _case("qwen2vl_batch_f16", "prune", dtype="f16", value_std=1.0, **qwen),
        _case("llava_batch_prob_f16", "prune", batch=64, mode="mean_prob", dtype="f16",
              value_std=1.0),
        # the largest: 4096-token images (documents, charts), both readings
        _case("hires_batch", "prune", **hires),
        _case("hires_batch_prob", "prune", mode="mean_prob", **hires),
        # dynamic resolution: Qwen2-VL images of 256 to 1600 tokens in one call
        _case("qwen2vl_ragged", "ragged", batch=32, heads=28, kv_heads=4, text=160, grid_h=40,
              grid_w=40, keep=355),
        # the progressive schedule 576 -> 122 -> 48 -> 42 with its compactions
        _case("llava_progressive", "progressive", batch=64, layers=3, keep=42),
    ]


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------

def _ragged_dims(c):
    """(grid_h, grid_w, num_text, keep) per image: sides from 40 % to all of the
    case's, text lengths from a fifth to all, the case's share of the tokens kept."""
    rng = random.Random(c["sizes_seed"])
    frac = c["keep"] / (c["grid_h"] * c["grid_w"])
    out = []
    for _ in range(c["batch"]):
        gh = rng.randint(max(c["cells"], 2 * c["grid_h"] // 5), c["grid_h"])
        gw = rng.randint(max(c["cells"], 2 * c["grid_w"] // 5), c["grid_w"])
        out.append((gh, gw, rng.randint(max(1, c["text"] // 5), c["text"]),
                    max(1, round(frac * gh * gw))))
    return out


def _budgets(c):
    """Kept tokens of the three progressive operations (576 -> 122 -> 48 -> 42)."""
    n, k = c["grid_h"] * c["grid_w"], c["keep"]
    k1 = max(k, round(n * 122 / 576))
    return [k1, max(k, min(k1, round(n * 48 / 576))), k]


def _image_dims(c):
    if c["entry"] == "ragged":
        return _ragged_dims(c)
    return [(c["grid_h"], c["grid_w"], c["text"], c["keep"])] * c["batch"]


HIDDEN = 4096


def work(case):
    c = case
    es = 4 if c["dtype"] == "f32" else 2
    L, H, G, D = c["layers"], c["heads"], c["kv_heads"], c["head_dim"]
    by = fl = 0.0
    if c["entry"] == "progressive":
        n = c["grid_h"] * c["grid_w"]
        for s, (m, k) in enumerate(zip([n] + _budgets(c)[:2], _budgets(c))):
            by += c["batch"] * ((H * c["text"] + G * m) * D * es + 20 * k)
            fl += _score_flops(c, 1, m, c["text"])
            if s > 0:                                   # the candidates' keys gathered
                by += c["batch"] * 2 * G * m * D * es
        by += c["batch"] * 2 * c["keep"] * HIDDEN * es
        return {"bytes": by, "flops": fl * c["batch"]}
    for gh, gw, nt, k in _image_dims(c):
        n = gh * gw
        by += L * (H * nt + G * n) * D * es + 16 * n + 4 * k
        fl += _score_flops(c, L, n, nt)
    return {"bytes": by, "flops": fl}


def _score_flops(c, layers, n, nt):
    per_row = 2.0 * layers * c["heads"] * c["head_dim"]
    if c["mode"] == "mean_prob":
        return per_row * nt * n
    return per_row * (n + nt / 2)


# ---------------------------------------------------------------------------
# further cases of the same ranges
# ---------------------------------------------------------------------------

def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49))))))


def draw(rng):
    """A case whose cost stays within the largest listed ones'."""
    most = {c["mode"]: work(c) for c in listed() if c["name"].startswith("hires")}
    while True:
        entry = rng.choice(["prune", "prune", "prune", "views", "ragged", "progressive"])
        gqa = entry == "ragged" or rng.random() < 0.45
        heads, kv = rng.choice([(28, 4), (16, 2), (32, 8), (12, 2)] if gqa
                               else [(32, 32), (32, 32), (16, 16), (40, 40), (4, 4)])
        side = lambda: _log_int(rng, 8, 64)                       # noqa: E731
        c = dict(entry=entry, batch=_log_int(rng, 1, 64), layers=rng.randint(1, 6), heads=heads,
                 kv_heads=kv, head_dim=rng.choice([64, 128, 128, 128]),
                 text=_log_int(rng, 8, 160), grid_h=side(), grid_w=side(), keep=0, cells=4,
                 lam=rng.choice([0.0, 0.1, 0.1, 0.5]),
                 mode=rng.choice(["mean_logit", "mean_prob"]),
                 dtype=rng.choice(["bf16", "bf16", "bf16", "f16", "f16", "f32"]),
                 value_std=rng.choice([0.0, 1.0]), sizes_seed=rng.randrange(1 << 30))
        if entry == "progressive":
            c["layers"] = 3
            c["mode"] = "mean_logit"
        n = c["grid_h"] * c["grid_w"]
        c["keep"] = max(4, round(n * rng.uniform(0.07, 0.35)))
        w = work(c)
        flops = w["flops"] * (8 if c["dtype"] == "f32" and c["mode"] == "mean_prob" else 1)
        if w["bytes"] <= most["mean_logit"]["bytes"] and flops <= most["mean_prob"]["flops"]:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _fill(c, q, k, gen, gh, gw):
    """q [B, H, N_T, d] and k [B, Hkv, N, d] (any strides) of one source layer get
    Gaussian elements, the salient tokens' keys shifted toward the mean query of
    their group."""
    std = c["value_std"] or 1.0 / math.sqrt(c["head_dim"])
    dev = q.device
    B, G, N, D = k.shape
    q.copy_(torch.randn(q.shape, generator=gen, device=dev) * std)
    x = torch.randn(k.shape, generator=gen, device=dev) * std
    cen = torch.rand((B, 3, 2), generator=gen, device=dev)
    row = (torch.arange(N, device=dev) // gw).float() / gh
    col = (torch.arange(N, device=dev) % gw).float() / gw
    d2 = ((row - cen[..., :1]) ** 2 + (col - cen[..., 1:]) ** 2).amin(1)          # [B, N]
    near = d2.topk(max(1, N // 20), dim=1, largest=False).indices
    sal = torch.zeros((B, N), device=dev).scatter_(1, near, 1.0)
    u = q.float().unflatten(1, (G, -1)).mean((2, 3))                              # [B, G, d]
    u = u / u.norm(dim=-1, keepdim=True).clamp_min(1e-20) * (1.5 * std)
    x += sal[:, None, :, None] * u[:, :, None, :]
    k.copy_(x)


def _inputs(case, seed):
    """The tensors of a case on the GPU, from the seed alone."""
    c, dev, dt = case, torch.device("cuda"), DTYPES[case["dtype"]]
    gen = torch.Generator(device=dev).manual_seed(2608 + int(seed))
    B, L, H, G, D = c["batch"], c["layers"], c["heads"], c["kv_heads"], c["head_dim"]
    gh, gw, nt = c["grid_h"], c["grid_w"], c["text"]
    n = gh * gw
    if c["entry"] == "ragged":
        dims = _ragged_dims(c)
        arr, qe, ke, _, _ = E.packed_images(dims, L, H, G, D)
        q = torch.empty(qe, device=dev, dtype=dt)
        k = torch.empty(ke, device=dev, dtype=dt)
        for im, (a, b, t, _) in zip(arr, dims):
            qi = q[im.q_offset:im.q_offset + L * H * t * D].view(L, H, t, D)
            ki = k[im.k_offset:im.k_offset + L * G * a * b * D].view(L, G, a * b, D)
            for l in range(L):
                _fill(c, qi[l:l + 1], ki[l:l + 1], gen, a, b)
        return {"q": q, "k": k, "images": arr, "dims": dims}
    if c["entry"] == "views":
        # token-major projections [B, T, H, d] and caches [B, Hkv, S, d] whose visual
        # tokens follow 35 system tokens and precede the text
        sys_tokens = 35
        ql = [torch.empty((B, nt, H, D), device=dev, dtype=dt).transpose(1, 2) for _ in range(L)]
        kl = [torch.zeros((B, G, sys_tokens + n + nt, D), device=dev, dtype=dt)[
            :, :, sys_tokens:sys_tokens + n] for _ in range(L)]
        for l in range(L):
            _fill(c, ql[l], kl[l], gen, gh, gw)
        return {"q": ql, "k": kl}
    if c["entry"] == "progressive":
        q = [torch.empty((B, 1, H, nt, D), device=dev, dtype=dt) for _ in range(L)]
        k = [torch.empty((B, 1, G, n, D), device=dev, dtype=dt) for _ in range(L)]
        for l in range(L):
            _fill(c, q[l][:, 0], k[l][:, 0], gen, gh, gw)
        hidden = torch.randn((B, 1, n, HIDDEN), generator=gen, device=dev).to(dt)
        return {"q": q, "k": k, "hidden": hidden}
    q = torch.empty((B, L, H, nt, D), device=dev, dtype=dt)
    k = torch.empty((B, L, G, n, D), device=dev, dtype=dt)
    for l in range(L):
        _fill(c, q[:, l], k[:, l], gen, gh, gw)
    return {"q": q, "k": k}


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    dev, n = torch.device("cuda"), case["grid_h"] * case["grid_w"]
    opt = dict(cells=c["cells"], lam=c["lam"], mode=c["mode"])
    s["case"], s["opt"] = c, opt
    if c["entry"] == "prune":
        s["call"] = E.Pruner(s["q"], s["k"], c["grid_h"], c["grid_w"], c["keep"], **opt)
        s["fused"] = torch.empty((c["batch"], n, 3), device=dev)
        s["prio"] = torch.empty((c["batch"], n), device=dev)
    elif c["entry"] == "ragged":
        code = {"bf16": 1, "f16": 2, "f32": 0}[c["dtype"]]
        p = E.RaggedPruner(s["images"], c["layers"], c["heads"], c["kv_heads"], c["head_dim"], dev,
                           code, **opt)
        s["call"] = p
        s["fused"] = torch.empty((p.tokens, 3), device=dev)
        s["prio"] = torch.empty(p.tokens, device=dev)
    elif c["entry"] == "progressive":
        cand, s["stages"] = n, []
        for l, keep in enumerate(_budgets(c)):
            k = s["k"][l][:, :, :, :cand].contiguous()           # for its shape
            s["stages"].append(E.StagePruner(s["q"][l], k, c["grid_h"], c["grid_w"], keep, **opt))
            cand = keep
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    if c["entry"] == "prune":
        keep = s["call"](s["q"], s["k"], s["fused"], s["prio"])
        return {"keep": keep, "fused": s["fused"], "prio": s["prio"]}
    if c["entry"] == "ragged":
        keep = s["call"](s["q"], s["k"], s["fused"], s["prio"])
        return {"keep": keep, "fused": s["fused"], "prio": s["prio"]}
    if c["entry"] == "views":
        keep, fused, prio = E.prune_views(s["q"], s["k"], c["grid_h"], c["grid_w"], c["keep"],
                                          want_fused=True, want_prio=True, **s["opt"])
        return {"keep": keep, "fused": fused, "prio": prio}
    pos = m = None
    for l, stage in enumerate(s["stages"]):
        k = s["k"][l]
        if l > 0:
            k = E.compact_tokens(k[:, 0], pos).unsqueeze(1)
        _, pos, m = stage(s["q"][l], k, cand_pos=pos, m_prev=m)
    return {"pos": pos, "m": m, "hidden": E.compact_tokens(s["hidden"], pos)}


# ---------------------------------------------------------------------------
# accuracy
# ---------------------------------------------------------------------------

def tolerance(case):
    # float32 sums of ~128 products behind logits of spread 1e-3 (standard recipe)
    # or 1, carried into masses of order 1e-4.  Measured against exact(): masses
    # within 2.3e-7, priorities within 7.3e-6; a rounding may swap two tokens at the
    # edge of an image's kept set
    return {"rel": 3e-5, "max": 2e-3, "differ": 0.01}


def _evidence64(c, q, k):
    """Eq. 1, 8-10 of one layer of one image in float64: rho and ebar [N]."""
    q, k = q.double(), k.double()
    H, N = q.shape[0], k.shape[1]
    k = k.repeat_interleave(H // k.shape[0], 0)
    scale = 1.0 / math.sqrt(q.shape[-1])
    if c["mode"] == "mean_logit":
        r = torch.softmax((k @ q.mean(1).unsqueeze(-1)).squeeze(-1) * scale, -1)
    else:
        r = torch.softmax(q @ k.transpose(1, 2).contiguous() * scale, -1).mean(1)
    x = N * r
    e = (x - 1) / (2 * (1 + x))
    ebar = e.mean(0)
    rho = (2 * ebar).abs() * (1 - 2 * (e - ebar).abs().mean(0))
    return rho, ebar


def _fuse64(m, rho, ebar):
    """One layer combined onto the mass m [N, 3] (or None): the mass, the conflict."""
    n = torch.stack([rho * (0.5 + ebar), rho * (0.5 - ebar), 1 - rho], -1)
    if m is None:
        return n, torch.zeros_like(rho)
    kk = m[:, 0] * n[:, 1] + m[:, 1] * n[:, 0]
    one = [m[:, i] * n[:, i] + m[:, i] * n[:, 2] + m[:, 2] * n[:, i] for i in (0, 1)]
    return torch.stack(one + [m[:, 2] * n[:, 2]], -1) / (1 - kk)[:, None], kk


def _select64(c, prio, pos, gh, gw, keep):
    """Eq. 20-23: the kept indices, ascending."""
    G = c["cells"]
    lam = float(torch.tensor(c["lam"], dtype=torch.float32))
    cell = (pos // gw) * G // gh * G + (pos % gw) * G // gw
    order = torch.sort(prio, stable=True).indices
    oc = cell[order].tolist()
    adj = (1 - lam) * prio + lam
    seen = set()
    for i, x in zip(order.tolist(), oc):
        if x not in seen:
            seen.add(x)
            adj[i] = (1 - lam) * prio[i]
    return torch.sort(torch.sort(adj, stable=True).indices[:keep]).values


def _image64(c, layers, gh, gw, keep):
    """The whole path of one image; layers: its (q, k) per source layer."""
    m = None
    for q, k in layers:
        m, kk = _fuse64(m, *_evidence64(c, q, k))
    prio = m[:, 1] * (1 - kk)
    pos = torch.arange(gh * gw, device=prio.device)
    return _select64(c, prio, pos, gh, gw, keep).int(), m, prio


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    B, L = c["batch"], c["layers"]
    if c["entry"] == "progressive":
        poss, ms, hid = [], [], []
        for b in range(B):
            pos = torch.arange(c["grid_h"] * c["grid_w"], device="cuda")
            m = None
            for l, keep in enumerate(_budgets(c)):
                m, kk = _fuse64(m, *_evidence64(c, s["q"][l][b, 0], s["k"][l][b, 0][:, pos]))
                idx = _select64(c, m[:, 1] * (1 - kk), pos, c["grid_h"], c["grid_w"], keep)
                pos, m = pos[idx], m[idx]
            poss.append(pos.int())
            ms.append(m)
            hid.append(s["hidden"][b][:, pos].double())
        return {"pos": torch.stack(poss), "m": torch.stack(ms), "hidden": torch.stack(hid)}
    out = []
    for b, (gh, gw, nt, keep) in enumerate(_image_dims(c)):
        if c["entry"] == "ragged":
            im, H, G, D = s["images"][b], c["heads"], c["kv_heads"], c["head_dim"]
            q = s["q"][im.q_offset:im.q_offset + L * H * nt * D].view(L, H, nt, D)
            k = s["k"][im.k_offset:im.k_offset + L * G * gh * gw * D].view(L, G, gh * gw, D)
        elif c["entry"] == "views":
            q, k = [t[b] for t in s["q"]], [t[b] for t in s["k"]]
        else:
            q, k = s["q"][b], s["k"][b]
        out.append(_image64(c, [(q[l], k[l]) for l in range(L)], gh, gw, keep))
    join = torch.cat if c["entry"] == "ragged" else torch.stack
    return {"keep": join([o[0] for o in out]), "fused": join([o[1] for o in out]),
            "prio": join([o[2] for o in out])}
