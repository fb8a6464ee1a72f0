"""Slices whose rows do not fill 256-row blocks: blocks with waves past the slice, and (where the library packs the heads)
blocks that hold the end of one head and the start of the next.  Against the fp64 oracle."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, max_abs, rel_l2, out_err, TOL_OUT, TOL_LSE, TOL_GRAD

pytestmark = pytest.mark.gpu


# rows 1, one wave short of / past a block; too few blocks for the packed form
@pytest.mark.parametrize("B,s,Hq,Hkv,causal", [(1, 1, 8, 1, True), (1, 31, 6, 2, True), (2, 33, 3, 1, False), (1, 225, 4, 1, True),
                                               (1, 257, 8, 1, True), (2, 290, 6, 2, True), (1, 513, 3, 3, True)])
@pytest.mark.parametrize("D", [128, 64])
def test_ragged_rows(B, s, Hq, Hkv, causal, D):
    N = s + 331
    plan = check_call(B, s, N, Hq, Hkv, causal, D, ((N - s, 0, N), (5, 3, N - 2)))
    assert plan.dq_items == plan.dq_ranges * Hq * B * -(-s // 256)


# as many blocks as compute units or more, a tenth of which packing saves, and few keys at the diagonal: 8 and 4 heads in a
# block, heads that start in the middle of a block, a last block with waves without rows, ten heads of two waves
@pytest.mark.parametrize("B,s,N,Hq,Hkv,causal,D", [(32, 1, 40, 8, 1, True, 64), (32, 31, 500, 8, 1, True, 128), (33, 33, 540, 8, 1, True, 64),
                                                  (22, 290, 300, 6, 2, False, 64), (11, 513, 600, 8, 1, False, 128), (26, 40, 700, 10, 1, True, 128)])
def test_rows_of_several_heads_in_one_block(B, s, N, Hq, Hkv, causal, D):
    plan = check_call(B, s, N, Hq, Hkv, causal, D, ((N - s, 0, N),) + (((N - s // 2, 0, N - 3),) if s > 1 else ()))
    blocks = Hkv * B * -(-(Hq // Hkv * -(-s // 32)) // 8)
    assert plan.dq_items == plan.dq_ranges * blocks < plan.dq_ranges * Hq * B * -(-s // 256)


def check_call(B, s, N, Hq, Hkv, causal, D, calls):
    """Forward and backward of the calls (offset, first key, end) against the oracle; the plan of the last backward."""
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    bits = {t: normal_bf16((B, n, h, D), 18, t) for t, n, h in (("q", s, Hq), ("do", s, Hq), ("k", N, Hkv), ("v", N, Hkv))}
    dev = {t: dev_bf16(x) for t, x in bits.items()}
    f64 = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    for off, a, b in calls:
        say("packed rows: B=%d s=%d heads %d/%d D=%d causal=%s keys [%d,%d) at %d" % (B, s, Hq, Hkv, D, causal, a, b, off))
        o, l = sp.slimpipe_attn_fwd(dev["q"], dev["k"], dev["v"], off, a, b, causal, scale, out_dtype=sp.F32)
        o_ref, l_ref = attn_fwd(f64["q"], f64["k"], f64["v"], off, a, b, causal, scale)
        torch.cuda.synchronize()
        assert out_err(host_f64(o), o_ref, False)[0] <= TOL_OUT and max_abs(host_f64(l), l_ref) <= TOL_LSE
        ob = o.to(torch.bfloat16)
        dk, dv = torch.zeros((B, N, Hkv, D), device="cuda:0"), torch.zeros((B, N, Hkv, D), device="cuda:0")
        dq = sp.slimpipe_attn_bwd(dev["q"], dev["k"], dev["v"], ob, dev["do"], l, off, a, b, dk, dv, causal, scale, dq_dtype=sp.F32,
                                  dkv_accumulate=False)
        torch.cuda.synchronize()
        refs = attn_bwd(f64["q"], f64["k"], f64["v"], host_f64(ob), f64["do"], host_f64(l), off, a, b, causal, scale)
        for name, x, r in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
            x = host_f64(x)
            assert np.isfinite(x).all(), name
            assert rel_l2(x, r) <= TOL_GRAD, (name, rel_l2(x, r))
        p = sp.make_params(dev["q"], dev["k"], ob, off, a, b, causal, scale)
        plan = sp.slimpipe_attn_bwd_plan(p, 1, sp.slimpipe_attn_workspace_bytes(p, True))
    return plan
