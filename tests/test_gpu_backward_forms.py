"""GPU parity of every form of the strict backward, at lengths off its tiles, with
the kernels that ran read from the profiler, so that a rule that retargets a
shape fails here instead of leaving a form untested."""
import numpy as np
import pytest

from forms import bwd_form
from gpu_util import normwise_error, oracle_reference, run_gpu, say, to_device
from workloads import make_inputs

pytestmark = pytest.mark.gpu

# Relative 2-norm: sums of up to 1,000 f32 terms round to about sqrt(1000) 2^-24 =
# 1.9e-6 of their size at most; measured 3e-7 to 8e-7.
REL = 2e-6

# (form, B, H, Lq, Lk, mode)
CASES = [
    # 64-key tiles: one a head, split queries, D in the kernel or before it
    ("fused", 2, 3, 33, 17, "causal"), ("fused", 1, 2, 300, 64, "full"),
    ("fused", 2, 5, 129, 130, "padded"), ("fused", 1, 9, 300, 500, "full"),
    # many short heads: tiles filled less than 60 %
    ("fused", 1, 600, 20, 20, "full"), ("fused", 1, 371, 25, 116, "full"),
    # 128-key tiles (causal, 512 or more of them), rows that see no key among them
    ("fused", 8, 8, 100, 1000, "causal"), ("fused", 8, 8, 129, 1037, "causal padded"),
    ("fused", 1, 520, 60, 66, "causal"),
    ("wide", 1, 260, 127, 127, "full"), ("wide", 2, 150, 130, 250, "causal"),
    ("wide", 4, 50, 200, 250, "padded"),
    ("pair", 1, 105, 125, 125, "full"), ("pair", 1, 50, 250, 300, "causal"),
    ("pair", 4, 26, 128, 120, "padded"),
]


def kernels_of(fn):
    import paper_2608_01563_amd as mg
    mg.mg_profile_enable(True)
    mg.mg_profile_reset()
    try:
        fn()
        return sorted(n.rsplit("_", 2)[0] for n in mg.mg_profile_collect())
    finally:
        mg.mg_profile_enable(False)


def inputs(B, H, Lq, Lk, mode, d):
    kl = None
    if "padded" in mode:
        kl = [max(1, (b + 1) * Lk // B) for b in range(B)]
    return make_inputs(B, H, Lq, d, causal="causal" in mode, seed=Lq + Lk + d, key_len=kl, Lk=Lk)


def check(x, form):
    got = {}
    ran = kernels_of(lambda: got.update(run_gpu(x)))
    assert ("attn_dkdvq" in ran) == (form == "fused"), ran
    ref = oracle_reference(x)
    for n in ("O", "LSE", "dQ", "dK", "dV"):
        fin = np.isfinite(ref[n])
        assert np.array_equal(got[n][~fin], ref[n][~fin]), n
        rel = np.linalg.norm(got[n][fin] - ref[n][fin]) / np.linalg.norm(ref[n][fin])
        assert rel <= REL, (n, rel)


@pytest.mark.parametrize("d", [32, 64])
@pytest.mark.parametrize("form,B,H,Lq,Lk,mode", CASES)
def test_form(gpu_lib, form, B, H, Lq, Lk, mode, d):
    say("backward form %s B=%d H=%d Lq=%d Lk=%d d=%d %s" % (form, B, H, Lq, Lk, d, mode))
    if d == 32 and form == "wide":
        H *= 2   # shorter workgroups: from twice as many
    assert bwd_form(B, H, Lq, Lk, d, mode.split()[0]) == form
    check(inputs(B, H, Lq, Lk, mode, d), form)


@pytest.mark.parametrize("form,B,H,Lq,Lk,mode", [
    ("pair", 1, 3, 33, 65, "causal"), ("pair", 2, 10, 257, 130, "full"),
    ("pair", 2, 16, 200, 200, "padded"), ("eight", 1, 150, 70, 90, "causal"),
    ("eight", 2, 40, 257, 200, "padded"),
])
def test_form_d128(gpu_lib, form, B, H, Lq, Lk, mode):
    say("backward form %s B=%d H=%d Lq=%d Lk=%d d=128 %s" % (form, B, H, Lq, Lk, mode))
    assert bwd_form(B, H, Lq, Lk, 128, mode) == form
    check(inputs(B, H, Lq, Lk, mode, 128), form)


@pytest.mark.parametrize("causal", [False, True])
def test_separate_passes_without_room_for_partials(gpu_lib, causal):
    """B2 H6 L1500 d64 takes the fused kernel with the caller's workspace; its 106
    MiB of partials exceed the static scratch, so the call without a workspace
    runs the separate passes.  Both sum 1,500 terms of each row in other orders:
    1500^0.5 2^-24 = 2.3e-6 of a row's size, entry by entry at most 1e-5."""
    import torch
    import paper_2608_01563_amd as mg
    say("no room for partials causal=%s" % causal)
    x = make_inputs(2, 6, 1500, 64, causal=causal, seed=5)
    Q, K, V, dO = (to_device(x, n) for n in ("Q", "K", "V", "dO"))
    assert mg.mg_attn_bwd_workspace_bytes(2, 6, 1500, 64, causal, "strict_f32") > 64 << 20
    O, LSE = mg.attention_forward(Q, K, V, causal=causal, scale=x.scale)
    ref = [torch.full_like(Q, float("nan")) for _ in range(3)]
    got = [torch.full_like(Q, float("nan")) for _ in range(3)]
    ran = kernels_of(lambda: mg.mg_attn_bwd_cross(Q, K, V, O, LSE, dO, *ref, causal=causal,
                                                  scale=x.scale))
    assert "attn_dkdvq" in ran, ran
    ran = kernels_of(lambda: mg.mg_attn_bwd_noalloc(Q, K, V, O, LSE, dO, *got, causal=causal,
                                                    scale=x.scale))
    assert ran == ["attn_dkdv", "attn_dq"], ran
    for n, a, b in zip(("dQ", "dK", "dV"), got, ref):
        e = normwise_error(a.double().cpu().numpy(), b.double().cpu().numpy())
        assert e <= 1e-5, (n, e)
