"""GPU parity of every form of the strict forward, at lengths off its tiles, and
the cost of short heads."""
import numpy as np
import pytest

from forms import fwd_form
from gpu_util import say, to_device, key_len_device, to_host
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# Relative 2-norm: sums of up to 600 f32 terms round to about sqrt(600) 2^-24 =
# 1.5e-6 of their size at most; measured 1e-7 to 6e-7.
REL = 2e-6

# (form, B, H, Lq, Lk, mode, head dimensions)
CASES = [
    ("few_wave", 1, 3, 1, 1, "full", (32, 64, 128)), ("few_wave", 2, 3, 40, 16, "full", (32, 64, 128)),
    ("few_wave", 1, 700, 33, 33, "causal", (32, 64, 128)),
    ("few_wave", 2, 400, 17, 50, "padded", (32, 64, 128)),
    ("few", 1, 2, 64, 64, "causal", (32, 64, 128)), ("few", 2, 5, 33, 17, "padded", (32, 64, 128)),
    ("few", 1, 40, 61, 61, "full", (32, 64, 128)), ("few", 2, 4, 100, 257, "causal", (32, 64, 128)),
    ("few_long", 1, 3, 16, 600, "full", (32, 64, 128)),
    ("rows32", 1, 90, 130, 130, "full", (32, 64)), ("rows32", 1, 128, 190, 257, "causal", (32, 64)), ("rows32_quad", 2, 8, 450, 450, "full", (32, 64)),
    ("rows64", 1, 1100, 61, 61, "full", (64,)), ("rows64", 1, 300, 300, 100, "full", (32,)),
    ("rows64", 1, 600, 60, 100, "padded", (128,)), ("rows64", 1, 700, 127, 99, "full", (32,)),
    ("rows64", 1, 70, 1030, 9, "full", (32, 64)),
    ("rows64_pair", 8, 8, 260, 260, "full", (32, 64)), ("rows64_pair", 1, 50, 190, 257, "full", (128,)), ("rows64_pair", 1, 64, 130, 130, "causal", (128,)),
    ("rows128", 8, 64, 270, 270, "causal", (32, 64)), ("rows128", 1, 130, 257, 257, "full", (128,)),
    ("rows128", 1, 1100, 110, 110, "full", (32, 64)),
    ("rows256", 1, 600, 257, 257, "causal", (128,)),
    # tiles that both sides fill
    ("rows128", 1, 257, 125, 127, "full", (32, 64)), ("rows128", 2, 64, 250, 190, "full", (32, 64)),
    ("rows32", 1, 520, 17, 1100, "full", (64,)), ("rows32", 8, 8, 254, 256, "causal", (32,)),
    ("rows32", 2, 32, 127, 128, "full", (64,)), ("rows32_quad", 1, 32, 255, 254, "full", (32, 64)),
]


@pytest.mark.parametrize("form,B,H,Lq,Lk,mode,d",
                         [c[:6] + (d,) for c in CASES for d in c[6]])
def test_form(gpu_lib, form, B, H, Lq, Lk, mode, d):
    import torch
    import paper_2608_01563_amd as mg
    say("forward form %s B=%d H=%d Lq=%d Lk=%d d=%d %s" % (form, B, H, Lq, Lk, d, mode))
    assert fwd_form(B, H, Lq, Lk, d, mode) == form
    kl = [max(1, (b + 1) * Lk // (B + 1)) for b in range(B)] if mode == "padded" else None
    x = make_inputs(B, H, Lq, d, causal=mode == "causal", seed=Lq + Lk + d, key_len=kl, Lk=Lk)
    Q, K, V = (to_device(x, n) for n in ("Q", "K", "V"))
    for b, n in enumerate(kl or []):   # rows past each key length take no part
        K[b, :, n:] = V[b, :, n:] = float("nan")
    O = torch.full_like(Q, float("nan"))
    LSE = torch.full(Q.shape[:3], float("nan"), device=Q.device)
    mg.mg_attn_fwd_cross(Q, K, V, O, LSE, key_len_device(x), causal=x.causal, scale=x.scale)
    S = x.scale * torch.matmul(Q.double(), torch.nan_to_num(K.double()).transpose(-1, -2).contiguous())
    j = torch.arange(Lk, device="cuda")
    if mode == "causal":
        S.masked_fill_(j[None, :] > torch.arange(Lq, device="cuda")[:, None] + Lk - Lq, -np.inf)
    if kl:
        S.masked_fill_(j >= key_len_device(x)[:, None, None, None], -np.inf)
    rL = torch.logsumexp(S, -1)
    rO = torch.matmul(torch.exp(S - rL[..., None]), torch.nan_to_num(V.double()))
    for n, g, r in (("O", O, rO), ("LSE", LSE, rL)):
        assert ((g.double() - r).norm() / r.norm()).item() <= REL, n


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("L", [20, 35, 55])
def test_short_heads_cost_no_more_than_long_ones(gpu_lib, L, d):
    """As many rows in heads of L as in heads of 256, with a fifth or less of the
    products, take no longer (with a workgroup of 128 or 256 rows per short head
    they took up to 2.2 times as long)."""
    import torch
    import paper_2608_01563_amd as mg
    say("short heads L=%d d=%d" % (L, d))

    def us(H, L):
        Q, K, V = (torch.randn(1, H, L, d, device="cuda") for _ in range(3))
        O, LSE = torch.empty_like(Q), torch.empty(1, H, L, device="cuda")
        best = np.inf
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                mg.mg_attn_fwd(Q, K, V, O, LSE, causal=False, scale=d ** -0.5)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert us(300 * 256 // L, L) <= 1.1 * us(300, 256)
