"""Work items handed out through the ticket counters, one for all or one per XCD (items that walk 3072 keys and more, at
least eight groups of query blocks with keys of their own): every row is computed, whatever the number of groups, against slices of
the same call small enough to run without counters."""
import math

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


# (batch, rows, prefix, q heads, kv heads, counters of the dq items: none (the one launch), one for all, one per XCD): 8 groups
# exactly, with heads that share keys, a count that is no multiple of 8, one block per group
@pytest.mark.parametrize("B,s,N,Hq,Hkv,counters", [(1, 2304, 2304, 32, 8, 0), (1, 4096, 4096, 32, 8, 8), (3, 1280, 1536, 21, 21, 1),
                                                   (3, 1280, 3328, 21, 21, 8), (1, 200, 456, 300, 300, 1), (1, 200, 3100, 300, 300, 8)])
def test_every_item_is_computed_once(B, s, N, Hq, Hkv, counters):
    import torch
    import paper_2504_14519_amd as sp
    D, scale, G = 64, 0.125, Hq // Hkv
    say("items by XCD: batch %d, %d rows on %d keys, %d/%d heads" % (B, s, N, Hq, Hkv))
    g = torch.Generator(device="cuda:0").manual_seed(5)
    mk = lambda n, h: torch.randn((B, n, h, D), device="cuda:0", generator=g).to(torch.bfloat16)
    q, do, k, v = mk(s, Hq), mk(s, Hq), mk(N, Hkv), mk(N, Hkv)
    ws = torch.empty(256, device="cuda:0", dtype=torch.uint8)              # counters, no key ranges
    o, l = sp.slimpipe_attn_fwd(q, k, v, N - s, 0, N, True, scale, workspace=ws)
    wsb = torch.full((2 * ((B * Hq * s * 4 + 255) // 256 * 256) + 256,), 0xff, device="cuda:0", dtype=torch.uint8)
    dk, dv = torch.zeros((B, N, Hkv, D), device="cuda:0"), torch.zeros((B, N, Hkv, D), device="cuda:0")
    dq = sp.slimpipe_attn_bwd(q, k, v, o, do, l, N - s, 0, N, dk, dv, True, scale, dkv_accumulate=False, workspace=wsb)
    torch.cuda.synchronize()
    plan = sp.slimpipe_attn_bwd_plan(sp.make_params(q, k, o, N - s, 0, N, True, scale), 1, wsb.numel())
    assert plan.dkdv_split == 1 and plan.dq_ranges == 1 and plan.dq_items > plan.compute_units      # (the forward's items are as many)
    assert (plan.one_launch, plan.dq_by_xcd) == {0: (1, 0), 1: (0, 0), 8: (0, 1)}[counters] and B * Hkv >= 8
    for h in range(0, Hkv, max(1, Hkv // 7)):       # one K/V head at a time: few items, no counters
        qs, ks = slice(h * G, (h + 1) * G), slice(h, h + 1)
        o1, l1 = sp.slimpipe_attn_fwd(q[:, :, qs], k[:, :, ks], v[:, :, ks], N - s, 0, N, True, scale)
        assert torch.equal(o[:, :, qs], o1) and torch.equal(l[:, qs], l1), h
        p1 = sp.make_params(q[:, :, qs], k[:, :, ks], o1, N - s, 0, N, True, scale)
        assert sp.slimpipe_attn_bwd_plan(p1, 1, 1 << 40).one_launch == 1
        w1 = torch.empty(2 * ((B * G * s * 4 + 255) // 256 * 256), device="cuda:0", dtype=torch.uint8)
        # (the key/value strides of the one-head views are those of the whole cache, and so are the accumulators')
        dkf, dvf = torch.zeros_like(dk), torch.zeros_like(dv)
        dq1 = sp.slimpipe_attn_bwd(q[:, :, qs], k[:, :, ks], v[:, :, ks], o[:, :, qs], do[:, :, qs], l[:, qs].contiguous(), N - s, 0, N,
                                   dkf[:, :, ks], dvf[:, :, ks], True, scale, dq=torch.zeros_like(q)[:, :, qs], dkv_accumulate=False, workspace=w1)
        torch.cuda.synchronize()
        assert torch.equal(dq[:, :, qs], dq1), h
        assert torch.equal(dk[:, :, ks], dkf[:, :, ks]) and torch.equal(dv[:, :, ks], dvf[:, :, ks]), h
    assert torch.isfinite(o.float()).all() and torch.isfinite(dq.float()).all() and torch.isfinite(dk).all() and torch.isfinite(dv).all()
