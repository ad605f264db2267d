"""Problems whose workgroups hold 2^32 threads and more in all: a grid's size in
threads wraps there, so they run as several grids."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,d,contract", [
    (1, (1 << 24) + 5, 32, "strict_f32"), (1, (1 << 24) + 5, 32, "accelerated"),
    (3, 5592406, 32, "fast_bf16"), ((1 << 23) + 5, 1, 128, "strict_f32"),
    (4099, 2049, 64, "strict_f32"),
])
def test_attention_of_one_row_heads(gpu_lib, B, H, d, contract):
    """Heads of one row and one key: O = V, LSE = scale q k, dV = dO and no other
    gradient (dP - D cancels to rounding).  Every fifth batch element, where there
    are several, has no key: zeros."""
    import torch
    import paper_2608_01563_amd as mg
    say("one-row heads B=%d H=%d d=%d %s" % (B, H, d, contract))
    dt = torch.bfloat16 if contract == "fast_bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(1)
    Q, K, V, dO = (torch.randn(B, H, 1, d, generator=g, device="cuda", dtype=dt) for _ in range(4))
    kl = None
    if B > 1:
        kl = torch.ones(B, dtype=torch.int32, device="cuda")
        kl[4::5] = 0
    O, dQ, dK, dV = (torch.full_like(Q, float("nan")) for _ in range(4))
    LSE = torch.full((B, H, 1), float("nan"), device="cuda")
    kw = dict(causal=False, scale=0.25, contract=contract)
    mg.mg_attn_fwd(Q, K, V, O, LSE, kl, **kw)
    mg.mg_attn_bwd(Q, K, V, O, LSE, dO, dQ, dK, dV, kl, **kw)
    seen = torch.ones(B, 1, 1, 1, device="cuda") if kl is None else (kl > 0).view(B, 1, 1, 1)
    # O is V to its operands' rounding (an f16 subnormal's step is 2^-24).  The
    # backward's P = exp(s - LSE) is off from 1 by s's error in both directions: two
    # sums of d products whose sizes add up to less than 64, each rounded 24 times
    # (2 24 64 2^-24 < 2^-12); f16 operands there, 64 2^-10; bf16's O and dV, 2^-8.
    eps = {"strict_f32": 2.0 ** -12, "accelerated": 2.0 ** -4, "fast_bf16": 2.0 ** -7}[contract]
    tiny = 2.0 ** -24 if contract == "accelerated" else 0.0
    assert ((O - V * seen).abs() <= 2.0 ** -8 * V.abs() + tiny).all()
    assert ((dV - dO * seen).abs() <= eps * dO.abs()).all()
    s = 0.25 * (Q.float() * K.float()).sum(-1)
    on = seen.bool().expand(B, H, 1, 1)[..., 0]
    assert (LSE[on] - s[on]).abs().max() <= eps
    assert torch.isneginf(LSE[~on]).all()
    # |dP - D| <= eps |dO| |V| <= eps * 128 * 36, times |Q| or |K| <= 6, scale
    bound = eps * 128 * 36 * 6 * 0.25
    for t in (dQ, dK):
        assert t.abs().max() <= bound   # NaN fails too
        assert (t[~on] == 0).all()


def test_convolution_of_many_pixels(gpu_lib):
    """One channel, 23,170 x 23,170 pixels (2 GiB a tensor), 1x1."""
    import torch
    import paper_2608_01563_amd as mg
    say("convolution 23170 x 23170")
    X = torch.ones(1, 23170, 23170, 1, device="cuda")
    dY = torch.arange(23170, device="cuda", dtype=torch.float32).view(1, 1, -1, 1).expand_as(X)
    dY = (dY % 8).contiguous()
    W = torch.full((1, 1, 1, 1), 2.0, device="cuda")
    dX, dW = mg.conv2d_backward(X, W, dY)
    assert torch.equal(dX, 2 * dY)
    ref = dY.double().sum().item()
    assert abs(dW.item() - ref) <= 1e-6 * ref
