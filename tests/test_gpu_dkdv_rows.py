"""dk and dv rows of the 256-key items, which leave through LDS as whole rows: ranges that begin and end inside a wave's 32 keys, rows of K, V, dk
and dv apart by odd multiples of 8 elements, added to and overwritten, items of one launch and items that a workgroup takes one after
the other; against the fp64 oracle, and nothing is written between the rows or outside the range."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, rel_l2, TOL_GRAD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,s,Hq,Hkv,N,off,b,e,causal,pad,chunk,one_launch", [
    (1, 70, 2, 1, 600, 530, 0, 600, True, 8, 0, 1),           # a last wave of 24 keys
    (2, 33, 4, 2, 700, 500, 37, 609, False, 24, 0, 1),        # a range that ends with one key of a wave
    (1, 96, 3, 3, 1024, 700, 303, 785, True, 40, 256, 1),     # ... begins and ends inside a wave of the chunked grid
    (4, 33, 44, 44, 300, 267, 0, 300, True, 8, 0, 0),         # 352 items: the workgroups take them in turn
    (4, 40, 80, 40, 512, 300, 45, 331, True, 24, 256, 0),
])
def test_rows_of_dk_and_dv(D, B, s, Hq, Hkv, N, off, b, e, causal, pad, chunk, one_launch):
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    say("rows of dk and dv: B=%d s=%d N=%d %d/%d D=%d [%d,%d) causal %d pad %d chunk %d" % (B, s, N, Hq, Hkv, D, b, e, causal, pad, chunk))
    bits = {t: normal_bf16((B, N if t in "kv" else s, Hkv if t in "kv" else Hq, D), 75, t) for t in ("q", "k", "v", "do")}
    r = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    q, do = dev_bf16(bits["q"]), dev_bf16(bits["do"])
    L = chunk if chunk else N

    def rows_apart(x, fill):                                  # [B, N, Hkv, D] as chunks of L rows that are Hkv * D + pad apart
        wide = [torch.full((B, L, Hkv * D + pad), fill, device="cuda:0", dtype=x.dtype) for _ in range(0, N, L)]
        views = [w[:, :, :Hkv * D].unflatten(2, (Hkv, D)) for w in wide]
        for i, v in enumerate(views):
            v.copy_(x[:, i * L:(i + 1) * L])
        return views, wide
    k, v = rows_apart(dev_bf16(bits["k"]), 100.0)[0], rows_apart(dev_bf16(bits["v"]), float("nan"))[0]
    o_ref, l_ref = attn_fwd(r["q"], r["k"], r["v"], off, b, e, causal, scale)
    out, lse = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16), torch.from_numpy(l_ref).to("cuda:0").float()
    _, dk_ref, dv_ref = attn_bwd(r["q"], r["k"], r["v"], host_f64(out), r["do"], l_ref, off, b, e, causal, scale)
    p = sp.make_params(q, torch.empty((B, N, Hkv, D), device="meta"), out, off, b, e, causal, scale)
    room = 2 * ((B * Hq * s * 4 + 255) // 256 * 256) + 256    # statistics and counters: no cuts, no small kernel
    plan, path = sp.slimpipe_attn_bwd_plan(p, len(k), room), sp.slimpipe_attn_call_path(p, True, len(k), room)
    assert plan.one_launch == one_launch and path.small == 0 and plan.dkdv_split == 1
    assert one_launch or plan.dkdv_items > plan.compute_units
    ws = torch.full((room,), 255, device="cuda:0", dtype=torch.uint8)
    old = [torch.randn((B, N, Hkv, D), generator=torch.Generator().manual_seed(t)).to("cuda:0") for t in (1, 2)]
    first = {}
    for add in (True, False, True):
        (dk, wide_k), (dv, wide_v) = rows_apart(old[0], 7.0), rows_apart(old[1], 7.0)
        sp.slimpipe_attn_bwd_chunked(q, k, v, out, do, lse, off, b, e, dk, dv, causal, scale, dq_dtype=sp.F32, dkv_accumulate=add, workspace=ws)
        torch.cuda.synchronize()
        for name, got, start, want, wide in (("dk", dk, old[0], dk_ref, wide_k), ("dv", dv, old[1], dv_ref, wide_v)):
            got = torch.cat(got, 1)
            assert torch.equal(got[:, :b], start[:, :b]) and torch.equal(got[:, e:], start[:, e:]), "keys outside the range keep what they held"
            assert all((w[:, :, Hkv * D:] == 7.0).all() for w in wide), "nothing is written between the rows"
            mine = host_f64(got[:, b:e]) - (host_f64(start[:, b:e]) if add else 0.0)
            assert np.isfinite(mine).all()
            err = rel_l2(mine, want[:, b:e])
            say("%s %s rel-L2 %.3e" % (name, "added" if add else "written", err))
            assert err <= TOL_GRAD, name
            if add:
                assert torch.equal(first.setdefault(name, got), got), "bit-reproducible"
