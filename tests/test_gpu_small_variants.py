"""The four ways of a small backward call of head_dim 64 (one or two key blocks an item, row statistics of its own or of the delta kernel), each
asked of the plan query, grouped heads, several sequences, no causal mask, an odd last block, a chunked range; against the fp64 oracle."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, rel_l2, TOL_GRAD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,s,N,Hq,Hkv,causal,b,e,chunk,blocks,own", [
    (3, 306, 1197, 6, 2, True, 0, 1197, 0, 2, 0),        # grouped heads, a last block of 13 keys
    (1, 498, 1773, 12, 4, False, 0, 1773, 0, 2, 0),      # no mask; an odd number of blocks
    (3, 230, 2656, 8, 1, False, 0, 2656, 0, 2, 0),
    (3, 354, 2560, 8, 2, True, 45, 2533, 256, 2, 0),     # ... of a chunked cache, a range that begins and ends inside a block
    (3, 79, 1626, 8, 2, False, 0, 1626, 0, 2, 1),
    (2, 227, 1286, 12, 4, True, 0, 1286, 0, 2, 1),
    (1, 109, 1815, 12, 4, False, 0, 1815, 0, 2, 1),
    (2, 161, 545, 6, 2, True, 0, 545, 0, 1, 1),
    (1, 300, 740, 8, 1, False, 0, 740, 0, 1, 0),
])
def test_ways_of_a_small_backward(B, s, N, Hq, Hkv, causal, b, e, chunk, blocks, own):
    import torch
    import paper_2504_14519_amd as sp
    D, off, scale = 64, N - s, 1.0 / math.sqrt(64)
    say("small backward: B=%d s=%d N=%d %d/%d causal %d [%d,%d) chunk %d, %d blocks, own statistics %d" % (B, s, N, Hq, Hkv, causal, b, e, chunk, blocks, own))
    bits = {t: normal_bf16((B, N if t in "kv" else s, Hkv if t in "kv" else Hq, D), 76, t) for t in ("q", "k", "v", "do")}
    r = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    dev = {t: dev_bf16(x) for t, x in bits.items()}
    dev["k"][:, e:], dev["v"][:, e:] = float("nan"), float("nan")          # what the cache holds behind the range is not read
    o_ref, l_ref = attn_fwd(r["q"], r["k"], r["v"], off, b, e, causal, scale)
    out, lse = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16), torch.from_numpy(l_ref).to("cuda:0").float()
    want = attn_bwd(r["q"], r["k"], r["v"], host_f64(out), r["do"], l_ref, off, b, e, causal, scale)
    p = sp.make_params(dev["q"], dev["k"], out, off, b, e, causal, scale)
    ws = torch.full((sp.slimpipe_attn_workspace_bytes(p, True),), 255, device="cuda:0", dtype=torch.uint8)
    n_chunks = N // chunk if chunk else 1
    plan = sp.slimpipe_attn_small_bwd_plan(p, n_chunks, ws.numel())
    assert (plan.small, plan.key_blocks, plan.own_statistics) == (1, blocks, own)
    cut = lambda x: [x[:, i:i + N // n_chunks].contiguous() for i in range(0, N, N // n_chunks)]
    res = []
    for add in (True, True, False):
        dk, dv = cut(torch.full((B, N, Hkv, D), 0.5, device="cuda:0")), cut(torch.full((B, N, Hkv, D), -0.25, device="cuda:0"))
        sp.slimpipe_attn_profile_enable(True)
        try:
            dq = sp.slimpipe_attn_bwd_chunked(dev["q"], cut(dev["k"]), cut(dev["v"]), out, dev["do"], lse, off, b, e, dk, dv, causal, scale,
                                              dq_dtype=sp.F32, dkv_accumulate=add, workspace=ws)
        finally:
            sp.slimpipe_attn_profile_enable(False)
        torch.cuda.synchronize()
        assert {kind for kind, (_, n) in sp.slimpipe_attn_profile_read().items() if n} == ({"bwd_both"} if own else {"delta", "bwd_both"})
        dk, dv = torch.cat(dk, 1), torch.cat(dv, 1)
        res.append((dq, dk, dv))
        for name, g, w, old in (("dq", dq, want[0], 0.0), ("dk", dk[:, b:e], want[1][:, b:e], 0.5), ("dv", dv[:, b:e], want[2][:, b:e], -0.25)):
            g = host_f64(g) - (old if add else 0.0)
            assert np.isfinite(g).all(), name
            err = rel_l2(g, w)
            say("%s rel-L2 %.3e" % (name, err))
            assert err <= TOL_GRAD, name
        for x, old in ((dk, 0.5), (dv, -0.25)):
            assert (x[:, :b] == old).all() and (x[:, e:] == old).all(), "keys outside the range keep what they held"
    assert all(torch.equal(x, y) for x, y in zip(res[0], res[1])), "bit-reproducible"
