"""The calls that a user of this package makes, as cases to be timed and compared.

A case is one call of a public entry point: a whole denoising step of a band
(`DiTStep.step`), its conditioning, one attention layer, one projection of a
block, or a U-Net band block.  `listed()` holds one case for each kind of
real use, `draw(rng)` gives more of the same ranges.  Sizes are those of
seeded_inputs/configs.py (the tiny fp32 model, DiT-S/2 at 256px, DiT-XL/2 at
1024px and 2048px, the U-Net stages) and generic ones between them.
"""
import math
import struct

import torch

DEV = "cuda:0"
T, BETA = 1000, (1e-4, 2e-2)
CLASSES, FREQ = 1000, 256
STD = 0.02                        # weights are N(0, 0.02^2)


# ---- the cases ---------------------------------------------------------------

def _step(name, blocks, hidden, heads, latent, cfg_batch, dtype, row_begin, rows, t, t_prev,
          refresh=1, eta=0.0):
    return {"name": name, "kind": "step", "blocks": blocks, "hidden": hidden, "heads": heads,
            "latent": latent, "cfg_batch": cfg_batch, "dtype": dtype, "row_begin": row_begin,
            "rows": rows, "t": t, "t_prev": t_prev, "refresh": refresh, "eta": eta}


def _attention(name, B, heads, d, n_q, n_kv, fresh_begin, n_fresh, dtype):
    return {"name": name, "kind": "attention", "B": B, "heads": heads, "head_dim": d, "n_q": n_q,
            "n_kv": n_kv, "fresh_begin": fresh_begin, "n_fresh": n_fresh, "dtype": dtype}


def _linear(name, M, K, N, epilogue, dtype):
    return {"name": name, "kind": "linear", "M": M, "K": K, "N": N, "epilogue": epilogue,
            "dtype": dtype}


def _conditioning(name, blocks, hidden, heads, cfg_batch, dtype, t):
    return {"name": name, "kind": "conditioning", "blocks": blocks, "hidden": hidden, "heads": heads,
            "cfg_batch": cfg_batch, "dtype": dtype, "t": t}


def _unet(name, side, channels, groups, out_channels, row_begin, rows, refresh):
    return {"name": name, "kind": "unet", "side": side, "channels": channels, "groups": groups,
            "out_channels": out_channels, "row_begin": row_begin, "rows": rows, "refresh": refresh}


def listed():
    return [
        # the smallest model, fp32, half of its rows: a step that is all launches and latency
        _step("step_tiny_f32", 2, 128, 4, 16, 1, "f32", 0, 4, 500, 250),
        # DiT-S/2 at 256px, an interior 40% band, no guidance: a small model on one of several devices
        _step("step_s2_256_band40", 12, 384, 6, 32, 1, "bf16", 5, 6, 500, 450),
        # DiT-XL/2 at 1024px, the 40% band with guidance: one device's share of a production sampler
        _step("step_xl1024_band40", 28, 1152, 16, 128, 2, "bf16", 0, 26, 780, 760),
        # attention of a slow device's 10% band at 1024px: few queries against every key of the image
        _attention("attn_xl1024_band10", 2, 16, 72, 384, 4096, 1920, 384, "bf16"),
        # attention of an eighth of a 2048px image: the longest key stream
        _attention("attn_xl2048_band12", 2, 16, 72, 2048, 16384, 0, 2048, "bf16"),
        # attention with 128-channel heads, the widest the entry point takes, a ragged number of queries
        _attention("attn_d128_ragged", 2, 8, 128, 1000, 4096, 1024, 1000, "bf16"),
        # MLP out-projection with gated residual, 40% band at 1024px
        _linear("fc2_xl1024_band40", 3328, 4608, 1152, 2, "bf16"),
        # MLP in-projection with GELU, 5/8 of a 2048px image: the largest single projection
        _linear("fc1_xl2048_band62", 20480, 1152, 4608, 1, "bf16"),
        # a projection of the fp32 mode (reference runs), ragged rows
        _linear("qkv_s2_f32_ragged", 1000, 384, 1152, 0, "f32"),
        # timestep and label conditioning of every block of DiT-XL/2: streams 0.45 GB of weights
        _conditioning("conditioning_xl", 28, 1152, 16, 2, "bf16", 780),
        # first U-Net stage at 1024px, the larger half of an uneven two-device split, refreshing
        _unet("unet_stage1_72rows", 128, 320, 32, 320, 56, 72, 1),
        # deepest U-Net stage, an interior eighth: few pixels, many channels
        _unet("unet_stage3_4rows", 32, 1280, 32, 1280, 14, 4, 1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed kinds' ranges."""
    kind = rng.choice(("step", "attention", "attention", "linear", "linear", "conditioning", "unet"))
    widths = ((128, 4), (384, 6), (768, 12), (1152, 16))
    if kind == "step":
        hidden, heads = rng.choice(widths)
        f32 = hidden <= 384 and rng.random() < 0.35
        R = rng.choice((8, 16, 24, 32) if f32 else (8, 16, 24, 32, 48, 64))
        rows = rng.randint(1, R)
        t = rng.randint(1, T - 1)
        c = _step("", rng.randint(2, 8), hidden, heads, 2 * R, rng.randint(1, 2), "f32" if f32 else "bf16",
                  rng.randint(0, R - rows), rows, t, rng.randint(-1, t - 1), rng.randint(0, 1),
                  rng.choice((0.0, 0.0, 0.5)))
    elif kind == "attention":
        d = rng.choice((32, 64, 64, 72, 72, 80, 96, 128))
        f32 = rng.random() < 0.25
        R = rng.choice((8, 16, 24, 32) if f32 else (8, 16, 24, 32, 48, 64, 96))
        heads = rng.randint(4, 16)
        rows, B = min(R, _log_int(rng, 1, R)), rng.randint(1, 2)
        if d not in (64, 72) or f32:   # no more of these than the listed ones cost
            R = min(R, 64)
            rows = min(rows, max(1, 32768 // (B * heads * R)), R)
        fresh = rng.random() < 0.7
        c = _attention("", B, heads, d, rows * R, R * R, R * rng.randint(0, R - rows) if fresh else 0,
                       rows * R if fresh else 0, "f32" if f32 else "bf16")
    elif kind == "linear":
        H = rng.choice(widths)[0]
        K, N, epi = rng.choice(((H, 3 * H, 0), (H, H, 2), (H, 4 * H, 1), (4 * H, H, 2)))
        f32 = rng.random() < 0.25
        c = _linear("", _log_int(rng, 32, 4096 if f32 else 20480), K, N, epi, "f32" if f32 else "bf16")
    elif kind == "conditioning":
        hidden, heads = rng.choice(widths)
        c = _conditioning("", rng.randint(2, 28), hidden, heads, rng.randint(1, 2),
                          "f32" if rng.random() < 0.25 else "bf16", rng.randint(0, T - 1))
    else:
        side = rng.choice((16, 24, 32, 48, 64, 96, 120, 128))
        C = rng.choice([c for c in (64, 128, 192, 320, 640, 1280) if c * side * side <= 6 << 20])
        rows = min(side, _log_int(rng, 2, side))
        c = _unet("", side, C, rng.choice((8, 32)), rng.choice((C, C, 320, 640)), rng.randint(0, side - rows), rows,
                  rng.randint(0, 1))
    del c["name"]
    return c


# ---- inputs --------------------------------------------------------------------

def _td(dtype):
    return torch.float32 if dtype == "f32" else torch.bfloat16


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _randn(g, shape, std=1.0, dtype="f32"):
    return (torch.randn(shape, generator=g, device=DEV) * std).to(_td(dtype))


class _Config:
    """The model shape that DiTStep takes."""

    def __init__(self, case):
        self.n_blocks, self.hidden, self.heads = case["blocks"], case["hidden"], case["heads"]
        self.mlp_hidden, self.latent = 4 * case["hidden"], case.get("latent", 16)
        self.in_ch = self.out_ch = 4
        self.patch, self.num_classes, self.freq_dim = 2, CLASSES, FREQ
        self.cfg_batch, self.dtype = case["cfg_batch"], case["dtype"]
        self.T, (self.beta_start, self.beta_end) = T, BETA
        self.R = self.latent // 2


def _weights(case, g):
    """[(name, device tensor)] of the model in the blob's order."""
    cfg = _Config(case)
    H, F, R = cfg.hidden, cfg.mlp_hidden, cfg.R
    # DiT's fixed 2-D sine-cosine position table
    w = 10000.0 ** (-torch.arange(H // 4, dtype=torch.float64, device=DEV) / (H // 4))
    p = torch.arange(R, dtype=torch.float64, device=DEV)
    i, j = (p[:, None].expand(R, R).reshape(-1, 1) * w, p[None, :].expand(R, R).reshape(-1, 1) * w)
    pos = torch.cat([j.sin(), j.cos(), i.sin(), i.cos()], 1)
    out = [("x_embedder.weight", (H, 16)), ("x_embedder.bias", (H,)), ("pos_embed", pos),
           ("t1.weight", (H, FREQ)), ("t1.bias", (H,)), ("t2.weight", (H, H)), ("t2.bias", (H,)),
           ("table", (CLASSES + 1, H))]
    for l in range(cfg.n_blocks):
        out += [("%d.ada.weight" % l, (6 * H, H)), ("%d.ada.bias" % l, (6 * H,)),
                ("%d.qkv.weight" % l, (3 * H, H)), ("%d.qkv.bias" % l, (3 * H,)),
                ("%d.proj.weight" % l, (H, H)), ("%d.proj.bias" % l, (H,)),
                ("%d.fc1.weight" % l, (F, H)), ("%d.fc1.bias" % l, (F,)),
                ("%d.fc2.weight" % l, (H, F)), ("%d.fc2.bias" % l, (H,))]
    out += [("final.ada.weight", (2 * H, H)), ("final.ada.bias", (2 * H,)),
            ("final.weight", (16, H)), ("final.bias", (16,))]
    return [(n, s.to(_td(cfg.dtype)) if torch.is_tensor(s) else _randn(g, s, STD, cfg.dtype)) for n, s in out]


def _blob(case, weights):
    """The weight blob (host bytes): a 256-byte header, then the tensors, each 256-byte aligned."""
    cfg = _Config(case)
    es = 4 if cfg.dtype == "f32" else 2
    offs, off = [], 256
    for _, w in weights:
        offs.append(off)
        off = (off + w.numel() * es + 255) // 256 * 256
    blob = torch.zeros(off, dtype=torch.uint8, device=DEV)
    hdr = struct.pack("<8sII10II", b"ORCHDIT1", 1, 0 if es == 4 else 1, cfg.n_blocks, cfg.hidden, cfg.heads,
                      cfg.mlp_hidden, 4, 4, 2, cfg.R, CLASSES, FREQ, len(weights))
    blob[:len(hdr)] = torch.tensor(list(hdr), dtype=torch.uint8, device=DEV)
    for o, (_, w) in zip(offs, weights):
        blob[o:o + w.numel() * es] = w.reshape(-1).view(torch.uint8)
    return blob.cpu().numpy()


def _inputs(case, seed):
    """The device tensors of one call, from the seed alone."""
    g = _gen(seed)
    k, dt = case["kind"], case.get("dtype")
    if k in ("step", "conditioning"):
        cfg = _Config(case)
        s = {"weights": _weights(case, g)}
        s["labels"] = [int(torch.randint(0, CLASSES, (1,), generator=g, device=DEV))] + [CLASSES] * (cfg.cfg_batch - 1)
        if k == "step":
            H, n_kv = cfg.hidden, cfg.R * cfg.R
            s["x"] = _randn(g, (4, cfg.latent, cfg.latent))
            s["z"] = _randn(g, (4, cfg.latent, cfg.latent)) if case["eta"] else None
            # the spread of a linear layer's output on unit-variance inputs
            s["kv"] = torch.empty((cfg.n_blocks, cfg.cfg_batch, 2 * n_kv * H), dtype=_td(dt), device=DEV)
            for l in range(cfg.n_blocks):
                s["kv"][l] = _randn(g, (cfg.cfg_batch, 2 * n_kv * H), STD * math.sqrt(H), dt)
        return s
    if k == "attention":
        B, h, d, nf = case["B"], case["heads"], case["head_dim"], case["n_fresh"]
        std = 0.68                  # Q, K and V of a layer at this initialisation
        return {"q": _randn(g, (B, h, case["n_q"], d), std, dt),
                "stale": _randn(g, (B, 2 * h * case["n_kv"] * d), std, dt),
                "fresh": _randn(g, (B, 2 * h * nf * d), std, dt) if nf else None}
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        s = {"A": _randn(g, (M, K), 1.0 if case["epilogue"] != 2 else 0.5, dt), "W": _randn(g, (N, K), STD, dt),
             "bias": _randn(g, (N,), STD)}
        if case["epilogue"] == 2:   # two guidance branches, gate rows of the adaLN vectors
            s["gate"] = _randn(g, (2, 6 * N), 0.3)
            s["h"] = _randn(g, (M, N))
        return s
    n, C, Co = case["side"], case["channels"], case["out_channels"]
    rb, re = case["row_begin"], case["row_begin"] + case["rows"]
    s = {"gamma": 1.0 + _randn(g, (C,), STD), "beta": _randn(g, (C,), STD),
         "weight": _randn(g, (Co, 3, 3, C), STD, "bf16"), "bias": _randn(g, (Co,), STD)}
    off = _randn(g, (C,), 0.5)      # group means that are not zero
    s["x"] = _randn(g, (re - rb, n, C)) + off
    old = _randn(g, (n, n, C)) + off
    s["sums"] = _row_sums(old, case["groups"]).float()
    y = (old - old.mean((0, 1))) * old.std((0, 1)).reciprocal()
    s["act"] = torch.nn.functional.silu(y * s["gamma"] + s["beta"]).bfloat16()
    return s


def _row_sums(x, groups):
    r, W, C = x.shape
    v = x.double().reshape(r, W, groups, C // groups)
    return torch.stack([v.sum((1, 3)), (v * v).sum((1, 3))], -1)


def _rows_per_batch(case):
    return (case["M"] + 1) // 2


# ---- the calls -------------------------------------------------------------------

def prepare(case, seed):
    from paper_2509_04719_amd import _lib as lib
    s = _inputs(case, seed)
    s.update(case=case, lib=lib)
    k, dt = case["kind"], lib.DTYPE_CODE[case.get("dtype", "bf16")]
    if k in ("step", "conditioning"):
        cfg = _Config(case)
        s["ctx"] = lib.DiTStep(cfg, _blob(case, s.pop("weights")))
        if k == "step":
            rows = case["rows"]
            s["eps"] = torch.empty((cfg.cfg_batch, 4, 2 * rows, cfg.latent), device=DEV)
            s["out"] = torch.empty((4, 2 * rows, cfg.latent), device=DEV)
        else:
            s["out"] = torch.empty((cfg.cfg_batch, 6 * cfg.hidden * cfg.n_blocks + 2 * cfg.hidden), device=DEV)
    elif k == "attention":
        B, h, d, n_q, n_kv = (case[i] for i in ("B", "heads", "head_dim", "n_q", "n_kv"))
        s["out"] = torch.empty((B, n_q, h * d), dtype=_td(case["dtype"]), device=DEV)
        need = lib.attention_workspace_bytes(B, h, n_q, n_kv, d, dt)
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV) if need else None
    elif k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        s["out"] = s["h"] if case["epilogue"] == 2 else torch.empty((M, N), dtype=_td(case["dtype"]), device=DEV)
        need = lib.linear_workspace_bytes(M, N, K, dt)
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV) if need else None
    else:
        s["shape"] = lib.UNetConvShape(case["side"], case["side"], case["channels"], case["groups"],
                                       case["out_channels"], 1e-5)
        s["ws"] = torch.empty(lib.unet_conv_workspace_bytes(s["shape"], case["rows"]), dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty((case["rows"], case["side"], case["out_channels"]), device=DEV)
    s["dt"] = dt
    return s


def run(s):
    case, lib, dt = s["case"], s["lib"], s["dt"]
    k = case["kind"]
    if k == "step":
        rb = case["row_begin"]
        s["ctx"].step(s["x"], rb, rb + case["rows"], case["t"], case["t_prev"], s["labels"], 1.5, s["kv"],
                      case["refresh"], s["out"], out_eps=s["eps"], z=s["z"], eta=case["eta"])
        return s["eps"], s["out"], s["kv"]
    if k == "conditioning":
        s["ctx"].conditioning(case["t"], s["labels"], s["out"])
        return s["out"]
    if k == "attention":
        B, h, d, n_q, n_kv, nf = (case[i] for i in ("B", "heads", "head_dim", "n_q", "n_kv", "n_fresh"))
        lib.attention(s["q"], s["stale"], 2 * h * n_kv * d, s["fresh"], 2 * h * nf * d, case["fresh_begin"], nf, B, h,
                      n_q, n_kv, d, s["out"], dt, workspace=s["ws"])
        return s["out"]
    if k == "linear":
        M, K, N, epi = (case[i] for i in ("M", "K", "N", "epilogue"))
        lib.linear(s["A"], M, K, s["W"], N, s["bias"], epi, s.get("gate"), 6 * N if epi == 2 else 0,
                   _rows_per_batch(case), s["out"], dt, workspace=s["ws"])
        return s["out"]
    rb = case["row_begin"]
    lib.unet_conv_band(s["shape"], rb, rb + case["rows"], s["x"], s["gamma"], s["beta"], s["weight"], s["bias"],
                       s["act"], s["sums"], case["refresh"], s["out"], s["ws"])
    return s["out"], s["act"], s["sums"]


# ---- what a call cannot do without -------------------------------------------------

def work(case):
    k = case["kind"]
    es = 4 if case.get("dtype") == "f32" else 2
    if k == "step":
        H, B, L, R = case["hidden"], case["cfg_batch"], case["blocks"], case["latent"] // 2
        n_q, n_kv = case["rows"] * R, R * R
        flops = B * (n_q * (L * (24 * H * H + 4 * n_kv * H) + 64 * H) + 12 * H * H * L + 4 * H * H) + 512 * H + 2 * H * H
        weights = L * 18 * H * H + 3 * H * H + (FREQ + 16 + 16) * H
        kv = L * B * 2 * (n_kv - n_q) * H + (L * B * 2 * n_q * H if case["refresh"] else 0)
        return {"bytes": (weights + kv) * es + 4 * n_q * H + 16 * n_q * (2 + B) * 4, "flops": flops}
    if k == "conditioning":
        H, B, L = case["hidden"], case["cfg_batch"], case["blocks"]
        n = 6 * H * L + 2 * H
        return {"bytes": (n * H + H * H + FREQ * H + B * H) * es + n * 4 * (B + 1), "flops": 2 * B * n * H}
    if k == "attention":
        B, H, n_q, n_kv = case["B"], case["heads"] * case["head_dim"], case["n_q"], case["n_kv"]
        return {"bytes": B * H * es * (2 * n_q + 2 * n_kv), "flops": 4 * B * n_q * n_kv * H}
    if k == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        out = M * N * 8 if case["epilogue"] == 2 else M * N * es
        return {"bytes": (M * K + N * K) * es + out + 4 * N, "flops": 2 * M * N * K}
    r, W, C, Co, G = (case[i] for i in ("rows", "side", "channels", "out_channels", "groups"))
    halo = (case["row_begin"] > 0) + (case["row_begin"] + r < W)
    n = r * W * (C + Co) * 4 + 9 * C * Co * 2 + halo * W * C * 2 + (W - r) * G * 8
    return {"bytes": n + (r * W * C * 2 + r * G * 8 if case["refresh"] else 0), "flops": 18 * r * W * C * Co}


def tolerance(case):
    # About four times the error against 64 bits: fp32 sums of up to 4608 products (2e-7 to 5e-7; 1e-7 in the fp32
    # residual stream); bf16 operands, probabilities and 16-bit results, rounded to 2^-9 (1e-3 to 3e-3), which the
    # whole step carries from each layer into the next.
    if case.get("dtype") == "f32" or case["kind"] == "conditioning":
        return {"rel": 2e-6}
    if case["kind"] == "linear":
        return {"rel": 1e-6 if case["epilogue"] == 2 else 4e-3}
    return {"rel": {"step": 8e-3, "attention": 1.2e-2, "unet": 4e-3}[case["kind"]]}


# ---- the same in 64 bits --------------------------------------------------------------

def _attend(q, K, V):
    """softmax(q K^T / sqrt(d)) V of one head, a few queries at a time.  q [n, d], K [m, d], V [d, m]."""
    out = torch.empty_like(q)
    c = max(1, (1 << 25) // K.shape[0])
    for i in range(0, q.shape[0], c):
        out[i:i + c] = torch.softmax(q[i:i + c] @ K.t() / math.sqrt(q.shape[1]), 1) @ V.t()
    return out


def _gelu(y):
    return torch.nn.functional.gelu(y, approximate="tanh")


def _adaln(case, w, t, labels):
    """The adaLN vectors of every block and the final layer, [B, 6 H L + 2 H]."""
    f = torch.exp(-math.log(10000.0) * torch.arange(FREQ // 2, dtype=torch.float64, device=DEV) / (FREQ // 2)) * t
    silu = torch.nn.functional.silu
    e = torch.cat([f.cos(), f.sin()])
    e = w["t2.weight"].double() @ silu(w["t1.weight"].double() @ e + w["t1.bias"].double()) + w["t2.bias"].double()
    c = silu(e + w["table"][labels].double())
    names = ["%d.ada" % l for l in range(case["blocks"])] + ["final.ada"]
    return torch.cat([c @ w[n + ".weight"].double().t() + w[n + ".bias"].double() for n in names], 1)


def _exact_step(case, s):
    cfg = _Config(case)
    w = dict(s["weights"])
    H, h, d, R, L, B = cfg.hidden, cfg.heads, cfg.hidden // cfg.heads, cfg.R, cfg.n_blocks, cfg.cfg_batch
    rb, r = case["row_begin"], case["rows"]
    n, n_kv, tok = r * R, R * R, slice(rb * R, (rb + r) * R)
    mod = _adaln(case, w, case["t"], s["labels"])
    x = s["x"].double()

    def lin(v, name):
        return v @ w[name + ".weight"].double().t() + w[name + ".bias"].double()

    def norm(v, shift, scale):
        return torch.nn.functional.layer_norm(v, (H,), eps=1e-6) * (1 + scale) + shift

    patches = x[:, 2 * rb:2 * (rb + r)].reshape(4, r, 2, R, 2).permute(1, 3, 0, 2, 4).reshape(n, 16)
    h0 = lin(patches, "x_embedder") + w["pos_embed"].double()[tok]
    kv = s["kv"].double()
    eps = torch.empty((B, 4, 2 * r, cfg.latent), dtype=torch.float64, device=DEV)
    for b in range(B):
        hb = h0.clone()
        for l in range(L):
            m = mod[b, 6 * H * l:6 * H * (l + 1)].reshape(6, H)
            qkv = lin(norm(hb, m[0], m[1]), "%d.qkv" % l).reshape(n, 3, h, d)
            K = kv[l, b, :n_kv * H].reshape(h, n_kv, d).clone()
            V = kv[l, b, n_kv * H:].reshape(h, d, n_kv).clone()
            K[:, tok] = qkv[:, 1].permute(1, 0, 2)
            V[:, :, tok] = qkv[:, 2].permute(1, 2, 0)
            if case["refresh"]:
                kv[l, b, :n_kv * H] = K.reshape(-1)
                kv[l, b, n_kv * H:] = V.reshape(-1)
            o = torch.cat([_attend(qkv[:, 0, i].contiguous(), K[i], V[i]) for i in range(h)], 1)
            hb = hb + m[2] * lin(o, "%d.proj" % l)
            hb = hb + m[5] * lin(_gelu(lin(norm(hb, m[3], m[4]), "%d.fc1" % l)), "%d.fc2" % l)
        y = lin(norm(hb, mod[b, -2 * H:-H], mod[b, -H:]), "final").reshape(r, R, 2, 2, 4)
        eps[b] = y.permute(4, 0, 2, 1, 3).reshape(4, 2 * r, cfg.latent)
    # the update x' = a x - b eps + c z of eta-DDIM on the linear-beta schedule
    ab = torch.cumprod(1 - torch.linspace(BETA[0], BETA[1], T, dtype=torch.float64), 0)
    s_, p = float(ab[case["t"]]), float(ab[case["t_prev"]]) if case["t_prev"] >= 0 else 1.0
    c = case["eta"] * math.sqrt((1 - p) / (1 - s_)) * math.sqrt(1 - s_ / p)
    bc = math.sqrt(p) * math.sqrt(1 - s_) / math.sqrt(s_) - math.sqrt(max(0.0, 1 - p - c * c))
    e = eps[0] if B == 1 else eps[1] + 1.5 * (eps[0] - eps[1])
    band = slice(2 * rb, 2 * (rb + r))
    out = math.sqrt(p / s_) * x[:, band] - bc * e
    if c:
        out = out + c * s["z"].double()[:, band]
    return eps, out, kv


def _exact_attention(case, s):
    B, h, d, n_q, n_kv, nf, fb = (case[i] for i in ("B", "heads", "head_dim", "n_q", "n_kv", "n_fresh", "fresh_begin"))
    out = torch.empty((B, n_q, h * d), dtype=torch.float64, device=DEV)
    for b in range(B):
        K = s["stale"][b, :h * n_kv * d].double().reshape(h, n_kv, d)
        V = s["stale"][b, h * n_kv * d:].double().reshape(h, d, n_kv)
        if nf:
            K[:, fb:fb + nf] = s["fresh"][b, :h * nf * d].double().reshape(h, nf, d)
            V[:, :, fb:fb + nf] = s["fresh"][b, h * nf * d:].double().reshape(h, d, nf)
        for i in range(h):
            out[b, :, i * d:(i + 1) * d] = _attend(s["q"][b, i].double(), K[i], V[i])
    return out


def _exact_unet(case, s):
    n, C, G, r, rb = (case[i] for i in ("side", "channels", "groups", "rows", "row_begin"))
    x, sums, act = s["x"].double(), s["sums"].double(), s["act"].double()
    fresh = _row_sums(s["x"], G)
    allsums = sums.clone()
    allsums[rb:rb + r] = fresh
    N = n * n * (C // G)
    mean = allsums[..., 0].sum(0) / N
    rstd = (allsums[..., 1].sum(0) / N - mean * mean + 1e-5).rsqrt()
    v = ((x.reshape(r, n, G, C // G) - mean[:, None]) * rstd[:, None]).reshape(r, n, C)
    v = torch.nn.functional.silu(v * s["gamma"].double() + s["beta"].double())
    pad = torch.zeros((r + 2, n + 2, C), dtype=torch.float64, device=DEV)
    pad[1:r + 1, 1:n + 1] = v
    for row, y in ((0, rb - 1), (r + 1, rb + r)):
        if 0 <= y < n:
            pad[row, 1:n + 1] = act[y]
    W = s["weight"].double()
    out = s["bias"].double().expand(r * n, -1).clone()
    for dy in range(3):
        for dx in range(3):
            out += pad[dy:dy + r, dx:dx + n].reshape(r * n, C) @ W[:, dy, dx].t()
    if case["refresh"]:
        act[rb:rb + r], sums[rb:rb + r] = v, fresh
    return out.reshape(r, n, -1), act, sums


def exact(case, seed):
    s = _inputs(case, seed)
    k = case["kind"]
    if k == "step":
        return _exact_step(case, s)
    if k == "conditioning":
        return _adaln(case, dict(s["weights"]), case["t"], s["labels"])
    if k == "attention":
        return _exact_attention(case, s)
    if k == "unet":
        return _exact_unet(case, s)
    y = s["A"].double() @ s["W"].double().t() + s["bias"].double()
    if case["epilogue"] == 1:
        return _gelu(y)
    if case["epilogue"] == 2:
        rows = torch.arange(case["M"], device=DEV) // _rows_per_batch(case)
        return s["h"].double() + s["gate"][:, :case["N"]].double()[rows] * y
    return y
