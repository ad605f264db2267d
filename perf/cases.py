"""The calls whose speed counts for a user of this library, and how each is
made, checked and priced.

A case is one pass over preallocated device buffers through the public entry
points: an attention training step (`mg_attn_fwd_cross`, then
`mg_attn_bwd_cross`), an attention forward alone (inference: prefill, or a
decode step of few query rows over a long key/value cache), or the backward of
the three convolutions of a ResNet bottleneck block (`mg_conv2d_bwd` each).
"""
import math

import torch

import paper_2608_01563_amd as mg


def _attn(name, B, H, Lq, Lk, d, contract, mask, step=True):
    """mask: "causal" (bottom-right aligned), "full", or "padded" (every batch
    element has its own key length)."""
    return {"name": name, "kind": "attn", "B": B, "H": H, "Lq": Lq, "Lk": Lk, "d": d,
            "contract": contract, "mask": mask, "step": step}


def _conv(name, N, size, cin, width, stride):
    """Bottleneck block: 1x1 cin -> width, 3x3 width -> width with the stride,
    1x1 width -> 4 width, on size x size pixels."""
    return {"name": name, "kind": "conv", "N": N, "size": size, "cin": cin, "width": width,
            "stride": stride}


def listed():
    return [
        # the smallest training step: one head, where launches and latency are all there is
        _attn("step tiny f32", 1, 1, 64, 64, 32, "strict_f32", "causal"),
        # a small model's layer
        _attn("step small f32", 4, 4, 256, 256, 64, "strict_f32", "causal"),
        # the ordinary training step of a decoder layer in the default contract
        _attn("step causal f32", 8, 8, 1024, 1024, 64, "strict_f32", "causal"),
        # an encoder's padded batch
        _attn("step padded f32", 16, 12, 512, 512, 64, "strict_f32", "padded"),
        # image positions attending to a short text context
        _attn("step cross f32", 4, 8, 1024, 77, 64, "strict_f32", "full"),
        # a speech encoder's 1,500 positions, a multiple of no tile
        _attn("step ragged f32", 2, 6, 1500, 1500, 64, "strict_f32", "full"),
        # wide heads
        _attn("step d128 f32", 2, 8, 1024, 1024, 128, "strict_f32", "causal"),
        # a long-context layer, the largest case
        _attn("step long bf16", 2, 16, 4096, 4096, 128, "fast_bf16", "causal"),
        # an ordinary layer in bf16, at a length off every tile
        _attn("step ragged bf16", 8, 8, 1000, 1000, 64, "fast_bf16", "causal"),
        # prefill of a prompt batch in the accelerated contract
        _attn("prefill accel", 8, 8, 1024, 1024, 64, "accelerated", "causal", step=False),
        # one decode step of a served batch, caches filled to different lengths
        _attn("decode bf16", 8, 16, 1, 4096, 128, "fast_bf16", "padded", step=False),
        # one ResNet-50 block's derivatives at batch 4 (14 x 14 stage)
        _conv("conv block", 4, 14, 1024, 256, 1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Credited operations of the largest case drawn, per contract: what the listed
# cases of that contract reach (the f32 matrix rate is a sixteenth of bf16's).
_MOST = {"strict_f32": 4.0e10, "accelerated": 4.0e10, "fast_bf16": 4.0e11}


def draw(rng):
    what = rng.random()
    if what < 0.15:   # a block of one of the four stages, 224-pixel images or odd-sized crops
        stage = rng.randrange(4)
        width = 64 << stage
        size = (56, 28, 14, 7)[stage] + rng.choice((0, 0, 1, 3))
        first = rng.random() < 0.3
        return _unnamed(_conv("", rng.choice((1, 2, 3, 4)), size * 2 if first and stage else size,
                              (2 * width if first and stage else 64 if first else 4 * width),
                              width, 2 if first and stage else 1))
    contract = rng.choice(("strict_f32", "strict_f32", "strict_f32", "fast_bf16", "fast_bf16",
                           "accelerated"))
    d = rng.choice((32, 64, 64, 128))
    if what < 0.30:   # decode: few rows over a long cache
        return _unnamed(_attn("", rng.choice((1, 2, 4, 8, 16)), rng.choice((4, 6, 8, 12, 16)),
                              rng.choice((1, 1, 1, 2, 4, 7, 16)), _log(rng, 256, 8192), d, contract,
                              "padded", step=False))
    step = rng.random() < 0.75
    mask = rng.choice(("causal", "causal", "full", "padded"))
    while True:
        B, H = rng.choice((1, 2, 3, 4, 8, 16)), rng.choice((1, 2, 4, 6, 8, 12, 16))
        Lq = _log(rng, 40, 4096)
        Lk = Lq
        if rng.random() < 0.2:   # cross-attention; causal only where every row sees a key
            Lk = _log(rng, 16, 2048)
            if mask == "causal":
                Lk = max(Lk, Lq)
        c = _unnamed(_attn("", B, H, Lq, Lk, d, contract, mask, step))
        if work(c)["flops"] <= _MOST[contract]:
            return c


def _unnamed(c):
    return {k: v for k, v in c.items() if k != "name"}


# ------------------------------------------------------------------ attention --
def _attn_inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.bfloat16 if c["contract"] == "fast_bf16" else torch.float32

    def normal(L):
        x = torch.randn(c["B"], c["H"], L, c["d"], generator=g, device="cuda")
        return x.to(dt)

    Q, K, V, dO = normal(c["Lq"]), normal(c["Lk"]), normal(c["Lk"]), normal(c["Lq"])
    kl = None
    if c["mask"] == "padded":   # a quarter to all of the keys
        kl = torch.randint(max(1, c["Lk"] // 4), c["Lk"] + 1, (c["B"],), generator=g,
                           device="cuda", dtype=torch.int32)
    return Q, K, V, dO, kl


def _prepare_attn(c, seed):
    Q, K, V, dO, kl = _attn_inputs(c, seed)
    s = {"case": c, "Q": Q, "K": K, "V": V, "kl": kl, "O": torch.empty_like(Q),
         "LSE": torch.empty(Q.shape[:3], dtype=torch.float32, device="cuda"),
         "kw": {"causal": c["mask"] == "causal", "scale": 1.0 / math.sqrt(c["d"]),
                "contract": c["contract"]}}
    if c["step"]:
        n = mg.mg_attn_bwd_cross_workspace_bytes(c["B"], c["H"], c["Lq"], c["Lk"], c["d"],
                                                 c["mask"] == "causal", c["contract"])
        s.update(dO=dO, dQ=torch.empty_like(Q), dK=torch.empty_like(K), dV=torch.empty_like(V),
                 ws=torch.empty(max(n, 1), dtype=torch.uint8, device="cuda"))
    return s


def _run_attn(s):
    mg.mg_attn_fwd_cross(s["Q"], s["K"], s["V"], s["O"], s["LSE"], s["kl"], **s["kw"])
    if not s["case"]["step"]:
        return {"O": s["O"], "LSE": s["LSE"]}
    mg.mg_attn_bwd_cross(s["Q"], s["K"], s["V"], s["O"], s["LSE"], s["dO"], s["dQ"], s["dK"],
                         s["dV"], s["kl"], workspace=s["ws"], **s["kw"])
    return {"O": s["O"], "LSE": s["LSE"], "dQ": s["dQ"], "dK": s["dK"], "dV": s["dV"]}


def _work_attn(c):
    Lq, Lk = c["Lq"], c["Lk"]
    if c["mask"] == "causal":
        full = max(0, min(Lq, Lk))   # the last `full` rows see keys; the last row sees all
        pairs = sum(Lk - i for i in range(full))
    elif c["mask"] == "padded":      # key lengths are uniform over a quarter to all
        pairs = Lq * Lk * 0.625
    else:
        pairs = Lq * Lk
    pairs *= c["B"] * c["H"]
    e = 2 if c["contract"] == "fast_bf16" else 4
    q = c["B"] * c["H"] * Lq * c["d"] * e
    k = c["B"] * c["H"] * Lk * c["d"] * e * (0.625 if c["mask"] == "padded" else 1)
    lse = c["B"] * c["H"] * Lq * 4
    if not c["step"]:
        return {"bytes": 2 * q + 2 * k + lse, "flops": 4 * c["d"] * pairs}
    return {"bytes": 4 * q + 4 * k + lse, "flops": 14 * c["d"] * pairs}


def _exact_attn(c, seed):
    Q, K, V, dO, kl = _attn_inputs(c, seed)
    B, H, Lq, Lk = c["B"], c["H"], c["Lq"], c["Lk"]
    scale = 1.0 / math.sqrt(c["d"])
    j = torch.arange(Lk, device="cuda")
    i = torch.arange(Lq, device="cuda")
    names = ("O", "LSE") + (("dQ", "dK", "dV") if c["step"] else ())
    out = {n: [] for n in names}
    for b in range(B):
        allowed = torch.ones(Lq, Lk, dtype=torch.bool, device="cuda")
        if c["mask"] == "causal":
            allowed = j[None, :] <= i[:, None] + (Lk - Lq)
        if kl is not None:
            allowed = allowed & (j[None, :] < kl[b])
        for h in range(H):
            q, k, v, go = (t[b, h].double() for t in (Q, K, V, dO))
            S = (scale * (q @ k.T)).masked_fill(~allowed, -math.inf)
            lse = torch.logsumexp(S, dim=1)
            P = torch.exp(S - lse.masked_fill(torch.isinf(lse), 0.0)[:, None])
            o = P @ v
            out["O"].append(o)
            out["LSE"].append(lse)
            if c["step"]:
                dS = P * (go @ v.T - (go * o).sum(dim=1, keepdim=True))
                out["dQ"].append(scale * (dS @ k))
                out["dK"].append(scale * (dS.T @ q))
                out["dV"].append(P.T @ go)
    return {n: torch.stack(t).reshape(B, H, *t[0].shape) for n, t in out.items()}


# ---------------------------------------------------------------- convolution --
def _conv_layers(c):
    """(size, C, K, R, stride, pad) of the block's three convolutions."""
    out = (c["size"] + 2 - 3) // c["stride"] + 1
    return [(c["size"], c["cin"], c["width"], 1, 1, 0),
            (c["size"], c["width"], c["width"], 3, c["stride"], 1),
            (out, c["width"], 4 * c["width"], 1, 1, 0)]


def _conv_inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    layers = []
    for size, C, K, R, stride, pad in _conv_layers(c):
        P = (size + 2 * pad - R) // stride + 1
        layers.append((normal(c["N"], size, size, C),
                       normal(K, R, R, C) * math.sqrt(2.0 / (R * R * C)),
                       normal(c["N"], P, P, K), (stride, stride), (pad, pad)))
    return layers


def _prepare_conv(c, seed):
    layers = []
    for X, W, dY, stride, pad in _conv_inputs(c, seed):
        n = mg.mg_conv2d_bwd_workspace_bytes(X.shape, W.shape, stride, pad)
        layers.append((X, W, dY, torch.empty_like(X), torch.empty_like(W), stride, pad,
                       torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")))
    return {"case": c, "layers": layers}


def _run_conv(s):
    out = []
    for X, W, dY, dX, dW, stride, pad, ws in reversed(s["layers"]):
        mg.mg_conv2d_bwd(X, W, dY, dX, dW, stride=stride, pad=pad, workspace=ws)
        out.append((dX, dW))
    return out


def _work_conv(c):
    flops = nbytes = 0
    for size, C, K, R, stride, pad in _conv_layers(c):
        P = (size + 2 * pad - R) // stride + 1
        flops += 4 * c["N"] * P * P * K * R * R * C
        nbytes += 4 * (2 * c["N"] * size * size * C + 2 * K * R * R * C + c["N"] * P * P * K)
    return {"bytes": nbytes, "flops": flops}


def _exact_conv(c, seed):
    out = []
    for X, W, dY, (st, _), (pad, _) in reversed(_conv_inputs(c, seed)):
        N, S, _, C = X.shape
        K, R = W.shape[0], W.shape[1]
        P = dY.shape[1]
        X, W, dY = X.double(), W.double(), dY.double().reshape(-1, K)
        Xp = torch.zeros(N, S + 2 * pad, S + 2 * pad, C, dtype=torch.float64, device="cuda")
        Xp[:, pad:pad + S, pad:pad + S] = X
        dXp, dW = torch.zeros_like(Xp), torch.zeros_like(W)
        for r in range(R):
            for s in range(R):
                rows, cols = slice(r, r + st * (P - 1) + 1, st), slice(s, s + st * (P - 1) + 1, st)
                dW[:, r, s] = dY.T @ Xp[:, rows, cols].reshape(-1, C)
                dXp[:, rows, cols] += (dY @ W[:, r, s]).reshape(N, P, P, C)
        out.append((dXp[:, pad:pad + S, pad:pad + S].contiguous(), dW))
    return out


# ----------------------------------------------------------------- interface --
def prepare(case, seed):
    mg.load_library()
    return _prepare_conv(case, seed) if case["kind"] == "conv" else _prepare_attn(case, seed)


def run(state):
    return _run_conv(state) if state["case"]["kind"] == "conv" else _run_attn(state)


def work(case):
    return _work_conv(case) if case["kind"] == "conv" else _work_attn(case)


def exact(case, seed):
    return _exact_conv(case, seed) if case["kind"] == "conv" else _exact_attn(case, seed)


def tolerance(case):
    # About four times the largest error of any output against 64 bits: f32
    # products and sums 4e-7 to 9e-7, f16 operands 4e-4 (outputs; gradients at
    # the rounded forward's outputs somewhat more), bf16 operands 2.5e-3.
    return {"rel": {"fast_bf16": 1e-2, "accelerated": 2e-3}.get(case.get("contract"), 4e-6)}
