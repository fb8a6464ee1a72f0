"""Backward calls whose gradients lie over their own out and lse, which are read before any gradient is written: small calls with and
without row statistics of their own, two key blocks an item, the 256-row items; against the fp64 oracle."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, rel_l2, TOL_GRAD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["bf16 dq over out", "float32 dq over out and lse", "dk over out, dv over lse", "dk and dv chunks over out and lse"])
@pytest.mark.parametrize("s,N,Hq,Hkv,D,small", [
    (300, 768, 4, 4, 64, 1),               # own statistics
    (512, 2048, 4, 4, 64, 1),              # ... and two key blocks an item
    (300, 1280, 8, 1, 64, 1),              # statistics of the delta kernel
    (257, 1280, 8, 1, 128, 1),
    (300, 768, 4, 4, 64, 0),               # 256-row items (the workspace holds the statistics alone)
])
def test_gradients_over_out_and_lse(s, N, Hq, Hkv, D, small, over):
    import torch
    import paper_2504_14519_amd as sp
    off, scale = N - s, 1.0 / math.sqrt(D)
    say("%s: s=%d N=%d %d/%d D=%d small %d" % (over, s, N, Hq, Hkv, D, small))
    bits = {t: normal_bf16((1, N if t in "kv" else s, Hkv if t in "kv" else Hq, D), 74, t) for t in ("q", "k", "v", "do")}
    r = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    q, k, v, do = (dev_bf16(bits[t]) for t in ("q", "k", "v", "do"))
    o_ref, l_ref = attn_fwd(r["q"], r["k"], r["v"], off, 0, N, True, scale)
    o_in, l_in = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16), torch.from_numpy(l_ref).to("cuda:0").float()
    want = attn_bwd(r["q"], r["k"], r["v"], host_f64(o_in), r["do"], l_ref, off, 0, N, True, scale)
    least = 2 * ((Hq * s * 4 + 255) // 256 * 256)
    p = sp.make_params(q, k, o_in, off, 0, N, True, scale)
    ws = torch.empty(sp.slimpipe_attn_workspace_bytes(p, True) if small else least, device="cuda:0", dtype=torch.uint8)
    assert sp.slimpipe_attn_call_path(p, True, N // 256 if "chunks" in over else 1, ws.numel()).small == small

    n_out, n_lse, n_kv, L = s * Hq * D, Hq * s, N * Hkv * D, 256
    assert n_kv * 4 >= n_out * 2 + 512 and N % L == 0
    res = []
    for _ in range(3):
        mem = torch.full((4 * (n_out + 2 * n_kv) + n_out * 2 + 8 * n_lse,), 255, device="cuda:0", dtype=torch.uint8)
        at = [0]

        def take(n, dtype):
            size = torch.empty((), dtype=dtype).element_size()
            x = mem[at[0]:at[0] + n * size].view(dtype)
            at[0] += (n * size + 255) // 256 * 256
            return x
        kw = dict(causal=True, scale=scale, dkv_accumulate=False, workspace=ws)
        # each gradient's memory, and out and lse where the case puts them
        dq_f32 = "float32 dq" in over
        dq = take(n_out, torch.float32 if dq_f32 else torch.bfloat16)
        dk, dv = take(n_kv, torch.float32), take(n_kv, torch.float32)
        own_out, own_lse = take(n_out, torch.bfloat16), take(n_lse, torch.float32)
        out, lse = own_out, own_lse
        if over == "bf16 dq over out":
            out = dq
        elif dq_f32:                                     # out in the first half, lse in the second
            out, lse = dq.view(torch.bfloat16)[:n_out], dq[n_out // 2:n_out // 2 + n_lse]
        else:
            out, lse = dk.view(torch.bfloat16)[64:64 + n_out], dv[n_kv - n_lse:]
        out, lse = out.view(1, s, Hq, D), lse.view(1, Hq, s)
        out.copy_(o_in)
        lse.copy_(l_in)
        dq, dk, dv = dq.view(1, s, Hq, D), dk.view(1, N, Hkv, D), dv.view(1, N, Hkv, D)
        kw.update(dq=dq, dq_dtype=sp.F32 if dq_f32 else sp.BF16)
        if "chunks" in over:
            cut = lambda x: [x[:, i:i + L] for i in range(0, N, L)]
            sp.slimpipe_attn_bwd_chunked(q, cut(k), cut(v), out, do, lse, off, 0, N, cut(dk), cut(dv), **kw)
        else:
            sp.slimpipe_attn_bwd(q, k, v, out, do, lse, off, 0, N, dk, dv, **kw)
        torch.cuda.synchronize()
        for name, g, w in zip(("dq", "dk", "dv"), (dq, dk, dv), want):
            g = host_f64(g)
            assert np.isfinite(g).all(), name
            err = rel_l2(g, w)
            say("%s rel-L2 %.3e" % (name, err))
            assert err <= TOL_GRAD, name
        res.append([x.clone() for x in (dq, dk, dv)])
    assert all(torch.equal(x, y) for other in res[1:] for x, y in zip(res[0], other)), "the same bits every time"


@pytest.mark.parametrize("s,N,Hq,Hkv", [(300, 768, 4, 4), (512, 2048, 4, 4)])
def test_statistics_come_from_the_delta_kernel_where_gradients_lie_over_them(s, N, Hq, Hkv):
    import torch
    import paper_2504_14519_amd as sp
    D, off = 64, N - s
    q, do, o = (torch.randn((1, s, Hq, D), device="cuda:0").to(torch.bfloat16) for _ in range(3))
    k, v = (torch.randn((1, N, Hkv, D), device="cuda:0").to(torch.bfloat16) for _ in range(2))
    lse, dk, dv = torch.full((1, Hq, s), 7.0, device="cuda:0"), torch.zeros((1, N, Hkv, D), device="cuda:0"), torch.zeros((1, N, Hkv, D), device="cuda:0")
    ws = torch.empty(sp.slimpipe_attn_workspace_bytes(sp.make_params(q, k, o, off, 0, N, True, None), True), device="cuda:0", dtype=torch.uint8)
    behind = torch.empty((2, 1, s, Hq, D), device="cuda:0", dtype=torch.bfloat16)
    behind[0] = o
    for out, dq, kinds in ((o, torch.empty_like(q), {"bwd_both"}), (behind[0], behind[1], {"bwd_both"}), (o, o, {"delta", "bwd_both"})):
        sp.slimpipe_attn_profile_enable(True)
        try:
            sp.slimpipe_attn_bwd(q, k, v, out, do, lse, off, 0, N, dk, dv, True, None, dq=dq, workspace=ws)
        finally:
            sp.slimpipe_attn_profile_enable(False)
        torch.cuda.synchronize()
        assert {kind for kind, (_, n) in sp.slimpipe_attn_profile_read().items() if n} == kinds
