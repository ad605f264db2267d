"""GPU parity of the few-rows forward (16 query rows per workgroup, the key
tiles dealt to its waves, value columns split over workgroups when there are
few), every contract, and of the query-stationary forwards at their tile edges
on grids large enough to reach them.

The few-rows cases cover one and several key tiles per wave, waves without a
tile, four and eight waves, one, two and four column splits, rows and keys off
the 16-row and 16-, 32- and 64-key tiles, all masks, and a padded tail of NaN.
"""
import numpy as np
import pytest

from gpu_util import TOL, TOL_ACCEL_ROUNDED, key_len_device, normwise_error, say, to_device, \
    to_host
from workloads import make_inputs

pytestmark = pytest.mark.gpu

CONTRACTS = ("strict_f32", "fast_bf16", "accelerated")


def check_forward(x, contract, poison=False):
    import torch
    import paper_2608_01563_amd as mg
    from oracle import oracle_forward, round_to_f16
    Q, K, V = (to_device(x, n) for n in ("Q", "K", "V"))
    if poison:   # rows past each key length hold NaN and take no part
        for b, n in enumerate(x.key_len):
            K[b, :, int(n):] = float("nan")
            V[b, :, int(n):] = float("nan")
    O = torch.full_like(Q, float("nan"))
    LSE = torch.full(Q.shape[:3], float("nan"), dtype=torch.float32, device=Q.device)
    mg.mg_attn_fwd_cross(Q, K, V, O, LSE, key_len_device(x), causal=x.causal, scale=x.scale,
                         contract=contract)
    rO, rL = oracle_forward(x.Q, x.K, x.V, x.causal, x.scale, key_len=x.key_len)
    e_o, e_l = normwise_error(to_host(O), rO), normwise_error(to_host(LSE), rL)
    assert e_o <= TOL[contract] and e_l <= TOL[contract], (e_o, e_l)
    if contract == "accelerated":
        rO, rL = oracle_forward(round_to_f16(x.Q), round_to_f16(x.K), round_to_f16(x.V), x.causal,
                                x.scale, key_len=x.key_len)
        e_o, e_l = normwise_error(to_host(O), rO), normwise_error(to_host(LSE), rL)
        assert e_o <= TOL_ACCEL_ROUNDED["O"] and e_l <= TOL_ACCEL_ROUNDED["LSE"], (e_o, e_l)


# (B, H, Lq, Lk, mode)
FEW = [
    (1, 2, 1, 1, "full"), (1, 2, 1, 33, "full"), (1, 2, 16, 1057, "causal"),
    (2, 3, 7, 64, "padded"), (2, 40, 16, 31, "causal"), (3, 100, 5, 47, "padded"),
    (1, 130, 3, 1100, "padded"), (1, 3, 250, 250, "causal"), (1, 2, 17, 15, "causal"),
]


@pytest.mark.parametrize("contract", CONTRACTS)
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,H,Lq,Lk,mode", FEW)
def test_few_rows(gpu_lib, B, H, Lq, Lk, mode, d, contract):
    say("few rows %s B=%d H=%d Lq=%d Lk=%d d=%d %s" % (contract, B, H, Lq, Lk, d, mode))
    kl = None
    if mode == "padded":
        kl = [max(1, (b + 1) * Lk // (B + 1)) for b in range(B)]
    x = make_inputs(B, H, Lq, d, causal=mode == "causal", contract=contract,
                    seed=7 * Lq + Lk + d, key_len=kl, Lk=Lk)
    check_forward(x, contract, poison=mode == "padded")


@pytest.mark.parametrize("contract", CONTRACTS)
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("Lq,Lk", [(63, 63), (65, 65), (127, 129), (128, 64), (193, 193)])
def test_many_rows(gpu_lib, Lq, Lk, causal, d, contract):
    """More than 512 blocks of 16 rows: the query-stationary forwards."""
    H = 513 // ((Lq + 15) // 16) + 1
    say("many rows %s H=%d Lq=%d Lk=%d d=%d causal=%s" % (contract, H, Lq, Lk, d, causal))
    x = make_inputs(1, H, Lq, d, causal=causal, contract=contract, seed=Lq + Lk + d, Lk=Lk,
                    key_len=None if causal else [Lk - 3])
    check_forward(x, contract)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("Lq,Lk,mode", [(800, 800, "causal"), (769, 801, "padded"),
                                        (830, 790, "causal")])
def test_bf16_two_group_backward(gpu_lib, Lq, Lk, mode, d):
    """Long chains on a small grid: the bf16 backward's two wave groups per
    workgroup, tiles whose second half is masked or past the end among them."""
    from gpu_util import compare, oracle_reference, run_gpu
    say("bf16 two groups Lq=%d Lk=%d d=%d %s" % (Lq, Lk, d, mode))
    x = make_inputs(2, 2, Lq, d, causal=mode == "causal", contract="fast_bf16", seed=Lq + d, Lk=Lk,
                    key_len=[Lk - 33, 65] if mode == "padded" else None)
    errs = compare(run_gpu(x), oracle_reference(x), "fast_bf16")
    assert max(errs.values()) <= TOL["fast_bf16"], errs


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("Lq,Lk,mode", [
    (1, 1, "full"), (32, 32, "causal"), (33, 33, "causal"), (33, 65, "causal"), (96, 64, "causal"),
    (97, 31, "padded"), (128, 33, "full"), (65, 97, "padded"), (40, 129, "causal"), (129, 96, "full"),
])
def test_bf16_dq_where_waves_see_nothing(gpu_lib, Lq, Lk, mode, d):
    """The bf16 dQ kernel leaves out the 32 keys that no row of a wave sees, and
    all keys for waves without rows: lengths around its 32-row and 32-key steps."""
    from gpu_util import compare, oracle_reference, run_gpu
    say("bf16 dQ cut Lq=%d Lk=%d d=%d %s" % (Lq, Lk, d, mode))
    x = make_inputs(2, 3, Lq, d, causal=mode == "causal", contract="fast_bf16", seed=Lq + Lk + d, Lk=Lk,
                    key_len=[Lk, max(1, Lk - 33)] if mode == "padded" else None)
    errs = compare(run_gpu(x), oracle_reference(x), "fast_bf16")
    assert max(errs.values()) <= TOL["fast_bf16"], errs
