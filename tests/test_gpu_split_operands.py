"""GPU parity of the strict-f32 kernels that run on split bf16 operands, and
their results for operands that the split cannot carry (infinities, NaN, and
finite values that round to an infinite bf16) or that it must scale (values
near the smallest normal number)."""
import numpy as np
import pytest

from forms import bwd_form, fwd_form
from gpu_util import oracle_reference, run_gpu, say, to_host
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# Relative 2-norm of the error: a product of split operands is within 2^-22 of
# the f32 one, sums of up to 200 terms round to about sqrt(200) 2^-24 = 8e-7;
# twice that for the chain of two products.
REL = 2e-6

# (B, H, Lq, Lk, mode): many heads, rows and keys off the 16-, 32-, 64- and
# 128-row tiles
LARGE = [
    (2, 260, 33, 33, "causal"), (2, 256, 130, 65, "causal"), (2, 256, 65, 193, "causal"),
    (4, 128, 97, 70, "padded"), (2, 260, 64, 64, "full"),
    # fewer, which two wave groups may take
    (1, 230, 50, 64, "causal"), (2, 115, 65, 33, "full"), (4, 60, 193, 100, "padded"),
    (1, 113, 130, 257, "causal"),
]


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,H,Lq,Lk,mode", LARGE)
def test_large_grids(gpu_lib, B, H, Lq, Lk, mode, d):
    say("split operands B=%d H=%d Lq=%d Lk=%d d=%d %s" % (B, H, Lq, Lk, d, mode))
    kl = [1 + (b * Lk) // (B - 1) if b < B - 1 else Lk for b in range(B)] if mode == "padded" \
        else None
    x = make_inputs(B, H, Lq, d, causal=mode == "causal", seed=Lq + Lk + d, key_len=kl, Lk=Lk)
    got, ref = run_gpu(x), oracle_reference(x)
    for n in ("O", "LSE", "dQ", "dK", "dV"):
        fin = np.isfinite(ref[n])
        assert np.array_equal(got[n][~fin], ref[n][~fin]), n
        rel = np.linalg.norm(got[n][fin] - ref[n][fin]) / np.linalg.norm(ref[n][fin])
        assert rel <= REL, (n, rel)


# (B, H, Lq, Lk, mode): heads of middle length on short and on long key sides
SMALL = [
    (2, 6, 1100, 1100, "causal"), (1, 8, 600, 301, "full"), (1, 8, 523, 33, "full"),
    (8, 8, 250, 250, "causal"), (8, 12, 150, 150, "padded"), (16, 9, 66, 61, "full"),
    (4, 8, 300, 127, "full"), (4, 8, 261, 129, "full"),
]


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("B,H,Lq,Lk,mode", SMALL)
def test_small_grids(gpu_lib, B, H, Lq, Lk, mode, d):
    test_large_grids(gpu_lib, B, H, Lq, Lk, mode, d)


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("H,Lq,Lk", [(8, 600, 301), (40, 257, 61)])
def test_small_grids_carry_infinities(gpu_lib, H, Lq, Lk, d):
    """An infinite value entry: its column is infinite, the rest is right."""
    import torch
    import paper_2608_01563_amd as mg
    say("split operands small grid, infinity, H=%d Lq=%d Lk=%d d=%d" % (H, Lq, Lk, d))
    g = torch.Generator().manual_seed(Lk)
    Q = torch.randn(1, H, Lq, d, generator=g)
    K, V = torch.randn(1, H, Lk, d, generator=g), torch.randn(1, H, Lk, d, generator=g)
    V[0, 1, 20, 5] = np.inf
    O, LSE = mg.attention_forward(Q.cuda(), K.cuda(), V.cuda(), causal=False, scale=d ** -0.5)
    S = d ** -0.5 * torch.matmul(Q.double(), K.double().transpose(-1, -2).contiguous())
    ref = torch.matmul(torch.softmax(S, -1), V.double())
    O = O.cpu().double()
    assert torch.isposinf(O[0, 1, :, 5]).all()
    O[0, 1, :, 5] = ref[0, 1, :, 5] = 0
    assert (O - ref).norm() / ref.norm() <= REL
    assert (LSE.cpu() - torch.logsumexp(S, -1)).abs().max() <= 1e-5


@pytest.mark.parametrize("B,H,Lq,Lk,d,mode", [
    (2, 6, 1500, 1500, 64, "full"), (1, 16, 1587, 1587, 32, "full"),   # key groups
    (2, 8, 1024, 1024, 128, "causal"), (8, 8, 1024, 1024, 64, "causal"),
    (2, 4, 5, 1364, 64, "full"), (2, 6, 1, 1521, 128, "full"),         # few rows
])
def test_lse_rounds_once(gpu_lib, B, H, Lq, Lk, d, mode):
    """LSE of long rows is within the rounding of its last operations: half an
    ulp of a value of [4, 8), 2^-22 at most and 2^-22 / sqrt(3) = 1.4e-7 on
    average, 2.3e-8 of a value of 6 and more; 2^-25 leaves room for the scores'
    own error.  Rounded at every step of (m + log2 l) ln 2 it is 5e-8."""
    import torch
    import paper_2608_01563_amd as mg
    say("LSE B=%d H=%d Lq=%d Lk=%d d=%d %s" % (B, H, Lq, Lk, d, mode))
    g = torch.Generator(device="cuda").manual_seed(Lq + Lk)
    Q, K, V = (torch.randn(B, H, L, d, generator=g, device="cuda") for L in (Lq, Lk, Lk))
    _, LSE = mg.attention_forward(Q, K, V, causal=mode == "causal", scale=d ** -0.5)
    S = d ** -0.5 * torch.matmul(Q.double(), K.double().transpose(-1, -2).contiguous())
    if mode == "causal":
        S += torch.full((Lq, Lk), -np.inf, dtype=torch.float64, device="cuda").triu(1 + Lk - Lq)
    ref = torch.logsumexp(S, -1)
    assert ((LSE.double() - ref).norm() / ref.norm()).item() <= 2.0 ** -25


def plain(Q, K, V, dO, scale):
    """The equations in f64 torch, infinities and NaN carried as they come."""
    import torch
    Q, K, V, dO = (t.double() for t in (Q, K, V, dO))
    S = scale * torch.matmul(Q, K.transpose(-1, -2).contiguous())
    P = torch.softmax(S, dim=-1)
    O = torch.matmul(P, V)
    dP = torch.matmul(dO, V.transpose(-1, -2).contiguous())
    dS = P * (dP - (dO * O).sum(-1, keepdim=True))
    return {"O": O, "LSE": torch.logsumexp(S, -1), "dQ": scale * torch.matmul(dS, K),
            "dK": scale * torch.matmul(dS.transpose(-1, -2).contiguous(), Q),
            "dV": torch.matmul(P.transpose(-1, -2).contiguous(), dO)}


# (B, H, L, d) without a mask: forward forms of 32, 64 and 256 rows with one, two
# and four key groups, backward forms wide, pair, fused (f32) and eight
FORMS = [(8, 64, 130, 64), (1, 105, 125, 64), (1, 8, 700, 64), (8, 64, 130, 32), (2, 40, 250, 32),
         (8, 64, 130, 128), (1, 40, 257, 128)]
# ... and causal: wide, pair, eight
CAUSAL_FORMS = [(8, 64, 130, 64), (1, 105, 125, 64), (2, 40, 250, 32), (8, 64, 130, 32),
                (8, 64, 130, 128), (1, 40, 257, 128)]
FORM_NAMES = [("rows64", "wide"), ("rows64_pair", "pair"), ("rows32_quad", "fused"),
              ("rows64", "wide"), ("rows32", "pair"), ("rows256", "eight"), ("rows64_pair", "pair")]


def test_forms_are_the_ones_named():
    for (B, H, L, d), names in zip(FORMS, FORM_NAMES):
        assert (fwd_form(B, H, L, L, d, "full"), bwd_form(B, H, L, L, d, "full")) == names
    for B, H, L, d in CAUSAL_FORMS:
        assert not fwd_form(B, H, L, L, d, "causal").startswith("few")
        assert bwd_form(B, H, L, L, d, "causal") != "fused"


@pytest.mark.parametrize("B,H,L,d", FORMS)
@pytest.mark.parametrize("what", ["Q", "K", "V", "dO"])
def test_small_operands_keep_their_bits(gpu_lib, what, B, H, L, d):
    """An operand of about 2^-120, whose lower parts would fall below bf16's
    smallest normal number, gives results as close as one of 1."""
    import torch
    import paper_2608_01563_amd as mg
    say("split operands, %s small, B=%d H=%d L=%d d=%d" % (what, B, H, L, d))
    g = torch.Generator(device="cuda").manual_seed(L + d)
    t = {n: torch.randn(B, H, L, d, generator=g, device="cuda") for n in ("Q", "K", "V", "dO")}
    t[what] *= 2.0 ** -120
    Q, K, V, dO = t["Q"], t["K"], t["V"], t["dO"]
    O, LSE = mg.attention_forward(Q, K, V, causal=False, scale=d ** -0.5)
    got = dict(zip(("dQ", "dK", "dV"),
                   mg.attention_backward(Q, K, V, O, LSE, dO, causal=False, scale=d ** -0.5)))
    got.update(O=O, LSE=LSE)
    ref = plain(Q, K, V, dO, d ** -0.5)
    for n, v in got.items():
        rel = ((v.double() - ref[n]).norm() / ref[n].norm()).item()
        assert rel <= REL, (n, rel)


@pytest.mark.parametrize("which", ["X", "W", "dY"])
@pytest.mark.parametrize("K", [36, 50])   # 16- and 4-byte loads
def test_small_operands_keep_their_bits_in_convolutions(gpu_lib, K, which):
    import torch
    import paper_2608_01563_amd as mg
    say("split operands convolution, %s small, K=%d" % (which, K))
    g = torch.Generator(device="cuda").manual_seed(K)
    t = {"X": torch.randn(2, 9, 9, K, generator=g, device="cuda"),
         "W": torch.randn(K, 3, 3, K, generator=g, device="cuda"),
         "dY": torch.randn(2, 9, 9, K, generator=g, device="cuda")}
    t[which] *= 2.0 ** -120
    got = mg.conv2d_backward(t["X"], t["W"], t["dY"], pad=(1, 1))
    x, w = (t[n].double().cpu().permute(0, 3, 1, 2).requires_grad_() for n in ("X", "W"))
    torch.nn.functional.conv2d(x, w, padding=1).backward(t["dY"].double().cpu().permute(0, 3, 1, 2))
    for n, v, r in zip(("dX", "dW"), got, (x.grad, w.grad)):
        r = r.permute(0, 2, 3, 1)
        rel = ((v.double().cpu() - r).norm() / r.norm()).item()
        assert rel <= REL, (n, rel)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what,value", [("V", np.inf), ("V", -np.inf), ("V", np.nan),
                                        ("dO", np.inf), ("dO", 3.4e38), ("V", 3.4e38),
                                        ("Q", np.nan), ("K", np.nan)])
def test_values_the_split_cannot_carry(gpu_lib, what, value, d):
    """One such value in one head: entries are finite, infinite or NaN where
    f32 arithmetic has them so, and the finite ones are right."""
    import torch
    import paper_2608_01563_amd as mg
    say("split operands %s = %s d=%d" % (what, value, d))
    H, L = 520, 70
    x = make_inputs(1, H, L, d, causal=False, seed=d, qkv_std=0.3)
    t = {n: torch.from_numpy(getattr(x, n).copy()) for n in ("Q", "K", "V", "dO")}
    t[what][0, 1, 37, 5] = value
    Q, K, V, dO = (t[n].cuda() for n in ("Q", "K", "V", "dO"))
    O, LSE = mg.attention_forward(Q, K, V, causal=False, scale=x.scale)
    dQ, dK, dV = mg.attention_backward(Q, K, V, O, LSE, dO, causal=False, scale=x.scale)
    got = {n: to_host(v)[0, :3] for n, v in (("O", O), ("LSE", LSE), ("dQ", dQ), ("dK", dK),
                                             ("dV", dV))}
    ref = plain(*(t[n][:, :3] for n in ("Q", "K", "V", "dO")), x.scale)
    for n, g in got.items():
        r = ref[n][0].numpy()
        with np.errstate(over="ignore"):
            r = r.astype(np.float32).astype(np.float64)   # overflows as f32 results do
        if what == "Q" or what == "K":
            if n == "LSE":
                continue   # a NaN row's LSE is reported as -inf
        if np.isnan(value) or np.isinf(value) or n == "O" or n == "dV":
            assert np.array_equal(np.isfinite(g), np.isfinite(r)), n
        # heads 0 and 2 hold ordinary values
        for h in (0, 2):
            rel = np.linalg.norm(g[h] - r[h]) / np.linalg.norm(r[h])
            assert rel <= REL, (n, h, rel)
        fin = np.isfinite(g[1]) & np.isfinite(r[1])
        if fin.any() and np.abs(value) != 3.4e38:
            assert np.max(np.abs(g[1][fin] - r[1][fin])) <= 1e-4 * max(1.0, np.max(np.abs(r[1][fin]))), n


@pytest.mark.parametrize("B,H,L,d", FORMS)
@pytest.mark.parametrize("what", ["V", "dO"])
def test_finite_values_above_the_split(gpu_lib, what, B, H, L, d):
    """3.4e38 rounds to an infinite bf16: the rows it reaches are recomputed in
    f32, and every output is finite and right.  Rows (keys) of up to 700 terms
    of one size round to at most 700 2^-24 = 4e-5 of their norm."""
    import torch
    import paper_2608_01563_amd as mg
    say("split operands %s = 3.4e38 B=%d H=%d L=%d d=%d" % (what, B, H, L, d))
    g = torch.Generator(device="cuda").manual_seed(L + d)
    t = {n: 0.2 * torch.randn(B, H, L, d, generator=g, device="cuda") for n in ("Q", "K", "V", "dO")}
    t[what][B - 1, 1, 37, 5] = 3.4e38
    Q, K, V, dO = t["Q"], t["K"], t["V"], t["dO"]
    O, LSE = mg.attention_forward(Q, K, V, causal=False, scale=d ** -0.5)
    got = dict(zip(("dQ", "dK", "dV"),
                   mg.attention_backward(Q, K, V, O, LSE, dO, causal=False, scale=d ** -0.5)))
    got.update(O=O, LSE=LSE)
    ref = plain(Q[-1:], K[-1:], V[-1:], dO[-1:], d ** -0.5)
    for n, v in got.items():
        assert torch.isfinite(v).all(), n
        v, r = v[-1, 1].double(), ref[n][0, 1]
        if n == "LSE":
            v, r = v[:, None], r[:, None]
        assert ((v - r).norm(dim=-1) <= 4e-5 * r.norm(dim=-1)).all(), n


@pytest.mark.parametrize("B,H,L,d", CAUSAL_FORMS)
@pytest.mark.parametrize("what,value", [("V", np.inf), ("V", np.nan), ("K", np.nan), ("K", np.inf)])
def test_masked_values_take_no_part(gpu_lib, what, value, B, H, L, d):
    """Under a causal mask an infinite or NaN key or value row j changes no row
    before j, tiles that row and j share included."""
    import torch
    import paper_2608_01563_amd as mg
    say("split operands causal %s = %s B=%d H=%d L=%d d=%d" % (what, value, B, H, L, d))
    g = torch.Generator(device="cuda").manual_seed(L + d)
    t = {n: torch.randn(B, H, L, d, generator=g, device="cuda") for n in ("Q", "K", "V", "dO")}

    def step(x):
        O, LSE = mg.attention_forward(x["Q"], x["K"], x["V"], causal=True, scale=d ** -0.5)
        dQ, _, dV = mg.attention_backward(x["Q"], x["K"], x["V"], O, LSE, x["dO"], causal=True,
                                          scale=d ** -0.5)
        return {"O": O, "LSE": LSE, "dQ": dQ, "dV": dV}

    clean = step(t)
    hit = {n: v.clone() for n, v in t.items()}
    j = L // 2 + 5
    hit[what][0, 1, j, 3] = value
    got = step(hit)
    if what == "V":   # reaches O's column 3 and no P
        assert not torch.isfinite(got["O"][0, 1, j:, 3]).any()
        got["O"][0, 1, j:, 3] = clean["O"][0, 1, j:, 3]
    else:
        assert not torch.isfinite(got["O"][0, 1, j:]).any(dim=-1).all()
        for n in ("O", "LSE"):
            got[n][0, 1, j:] = clean[n][0, 1, j:]
        got["dV"][0, 1] = clean["dV"][0, 1]
    got["dQ"][0, 1, j:] = clean["dQ"][0, 1, j:]
    for n in got:   # recomputed rows sum in another order
        assert torch.allclose(got[n], clean[n], rtol=1e-5, atol=2e-6 * clean[n].abs().max().item(),
                              equal_nan=False), n


def gpu_us(fn):
    import torch
    fn()
    best = np.inf
    for _ in range(3):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b))
    return best


@pytest.mark.parametrize("what", ["all", "Q", "V", "dO"])
@pytest.mark.parametrize("d", [64, 128])
def test_a_diverged_step_stays_bounded(gpu_lib, d, what):
    """A step whose inputs are NaN, or hold one NaN a head, takes at most eight
    times a finite one's time (measured 1.1 to 3; a row at a time it was 15 to 90)."""
    import torch
    import paper_2608_01563_amd as mg
    say("diverged step %s d=%d" % (what, d))
    B, H, L = (8, 8, 1024) if d == 64 else (2, 8, 1024)
    g = torch.Generator(device="cuda").manual_seed(1)
    t = {n: torch.randn(B, H, L, d, generator=g, device="cuda") for n in ("Q", "K", "V", "dO")}

    def step():
        O, LSE = mg.attention_forward(t["Q"], t["K"], t["V"], causal=True, scale=d ** -0.5)
        mg.attention_backward(t["Q"], t["K"], t["V"], O, LSE, t["dO"], causal=True, scale=d ** -0.5)

    finite = gpu_us(step)
    for n in t if what == "all" else (what,):
        t[n][:, :, slice(None) if what == "all" else L // 2, :] = np.nan
    assert gpu_us(step) <= 8 * finite


@pytest.mark.parametrize("what", ["all", "X", "W", "dY"])
def test_a_diverged_convolution_stays_bounded(gpu_lib, what):
    import torch
    import paper_2608_01563_amd as mg
    say("diverged convolution %s" % what)
    g = torch.Generator(device="cuda").manual_seed(1)
    t = {"X": torch.randn(4, 28, 28, 128, generator=g, device="cuda"),
         "W": torch.randn(128, 3, 3, 128, generator=g, device="cuda"),
         "dY": torch.randn(4, 28, 28, 128, generator=g, device="cuda")}
    dX, dW = torch.empty_like(t["X"]), torch.empty_like(t["W"])
    ws = torch.empty(mg.mg_conv2d_bwd_workspace_bytes(dX.shape, dW.shape, (1, 1), (1, 1)),
                     dtype=torch.uint8, device="cuda")

    def step():
        mg.mg_conv2d_bwd(t["X"], t["W"], t["dY"], dX, dW, stride=(1, 1), pad=(1, 1), workspace=ws)

    finite = gpu_us(step)
    for n in t if what == "all" else (what,):
        if what == "all":
            t[n].fill_(np.nan)
        else:
            t[n][1, 1, 2, 3] = np.nan
    assert gpu_us(step) <= 8 * finite


@pytest.mark.parametrize("which", ["X", "W", "dY"])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_convolution_carries_infinities(gpu_lib, which, value):
    """A value that the split cannot carry changes the outputs it reaches in
    the equations and no others (3x3, stride 1, padding 1; channels 20 and 36
    so that tiles end inside)."""
    import torch
    import paper_2608_01563_amd as mg
    say("split operands convolution %s = %s" % (which, value))
    g = torch.Generator().manual_seed(3)
    X, W = torch.randn(2, 9, 9, 20, generator=g), torch.randn(36, 3, 3, 20, generator=g)
    dY = torch.randn(2, 9, 9, 36, generator=g)
    clean = mg.conv2d_backward(X.cuda(), W.cuda(), dY.cuda(), pad=(1, 1))
    t = {"X": X, "W": W, "dY": dY}[which]
    t[(1, 4, 5, 3) if which != "W" else (5, 1, 2, 3)] = value
    dX, dW = mg.conv2d_backward(X.cuda(), W.cuda(), dY.cuda(), pad=(1, 1))
    hit = {"dX": torch.zeros(dX.shape, dtype=torch.bool), "dW": torch.zeros(dW.shape, dtype=torch.bool)}
    if which == "X":       # dW[:, r, s, 3] through dY[1, 5 - r, 6 - s]
        hit["dW"][:, :, :, 3] = True
    elif which == "W":     # dX[n, h, w, 3] where output (h, w - 1) exists
        hit["dX"][:, :, 1:, 3] = True
    else:                  # dX[1, 3:6, 4:7], dW[3]
        hit["dX"][1, 3:6, 4:7] = True
        hit["dW"][3] = True
    for n, got, ref in (("dX", dX.cpu(), clean[0].cpu()), ("dW", dW.cpu(), clean[1].cpu())):
        assert not torch.isfinite(got[hit[n]]).any(), n
        rest = ~hit[n]
        assert torch.isfinite(got[rest]).all(), n
        assert torch.allclose(got[rest], ref[rest], rtol=1e-5, atol=1e-4), n
