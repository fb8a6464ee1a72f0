"""Row statistics (dO . O and lse) of small backward calls, worked out by the items themselves or by the delta kernel: both sides of the line
between the two at head_dim 64, ragged tiles, `out` and `d_out` with rows apart, rows that see no key; against the fp64 oracle."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, rel_l2, TOL_GRAD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,N,Hq,Hkv,off,b,launches_delta", [
    (192, 500, 8, 1, 308, 0, False),       # 6 query tiles x 8 heads: 6 steps of a wave
    (193, 500, 8, 1, 307, 0, True),        # 7 steps
    (300, 700, 4, 4, 400, 0, False),       # a last tile of 12 rows, fewer than eight tiles for most waves
    (257, 513, 8, 2, 130, 200, False),     # the first 70 rows see no key of the range; a last tile of one row
    (257, 513, 8, 1, 130, 200, True),
])
def test_statistics_of_small_calls(s, N, Hq, Hkv, off, b, launches_delta):
    import torch
    import paper_2504_14519_amd as sp
    B, D = 1, 64
    scale = 1.0 / math.sqrt(D)
    say("small backward statistics: s=%d N=%d %d/%d off=%d from key %d" % (s, N, Hq, Hkv, off, b))
    bits = {t: normal_bf16((B, N if t in "kv" else s, Hkv if t in "kv" else Hq, D), 72, t) for t in ("q", "k", "v", "do")}
    r = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    dev = {t: dev_bf16(x) for t, x in bits.items()}

    def rows_apart(x, pad):
        wide = torch.full((B, s, Hq * D + pad), float("nan"), device="cuda:0", dtype=x.dtype)
        view = wide[:, :, :Hq * D].unflatten(2, (Hq, D))
        view.copy_(x)
        return view
    o_ref, l_ref = attn_fwd(r["q"], r["k"], r["v"], off, b, N, True, scale)
    out, do = rows_apart(torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16), 24), rows_apart(dev["do"], 40)
    lse = torch.from_numpy(l_ref).to("cuda:0").float()
    want = attn_bwd(r["q"], r["k"], r["v"], host_f64(out), r["do"], l_ref, off, b, N, True, scale)
    p = sp.make_params(dev["q"], dev["k"], out, off, b, N, True, scale)
    ws = torch.full((sp.slimpipe_attn_workspace_bytes(p, True),), 255, device="cuda:0", dtype=torch.uint8)
    assert sp.slimpipe_attn_call_path(p, True, 1, ws.numel()).small == 1
    dk, dv = torch.zeros((B, N, Hkv, D), device="cuda:0"), torch.zeros((B, N, Hkv, D), device="cuda:0")
    sp.slimpipe_attn_profile_enable(True)
    try:
        dq = sp.slimpipe_attn_bwd(dev["q"], dev["k"], dev["v"], out, do, lse, off, b, N, dk, dv, True, scale, dq_dtype=sp.F32, workspace=ws)
    finally:
        sp.slimpipe_attn_profile_enable(False)
    torch.cuda.synchronize()
    launched = {kind for kind, (_, n) in sp.slimpipe_attn_profile_read().items() if n}
    assert launched == ({"delta", "bwd_both"} if launches_delta else {"bwd_both"})
    for name, g, w in zip(("dq", "dk", "dv"), (dq, dk, dv), want):
        g = host_f64(g)
        assert np.isfinite(g).all(), name
        err = rel_l2(g, w)
        say("%s rel-L2 %.3e" % (name, err))
        assert err <= TOL_GRAD, name


# Calls of more dk/dv items than fit beside the dq items in one round, so that an item owns two blocks of 32 keys
@pytest.mark.parametrize("s,N,off,b,e,chunk", [
    (512, 2048, 1536, 0, 2048, 0),
    (500, 2010, 1510, 0, 2010, 0),         # 63 key blocks a head: the last item has one, of 26 keys
    (300, 2600, 2200, 37, 2500, 0),        # a range that begins and ends inside a block; 77 blocks
    (300, 2560, 2200, 37, 2500, 256),      # the same on the grid of a chunked cache
    (600, 2048, 1500, 0, 2048, 0),         # 19 query tiles; the last rows see every key
    (512, 2048, 1400, 0, 2048, 0),         # keys that no row sees
])
def test_two_key_blocks_an_item(s, N, off, b, e, chunk):
    import torch
    import paper_2504_14519_amd as sp
    B, H, D = 1, 4, 64
    scale = 1.0 / math.sqrt(D)
    say("small backward, two key blocks: s=%d N=%d off=%d [%d,%d) chunk %d" % (s, N, off, b, e, chunk))
    bits = {t: normal_bf16((B, N if t in "kv" else s, H, D), 73, t) for t in ("q", "k", "v", "do")}
    r = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    dev = {t: dev_bf16(x) for t, x in bits.items()}
    dev["k"][:, e:], dev["v"][:, e:] = float("nan"), float("nan")          # what the cache holds behind the range is not read
    o_ref, l_ref = attn_fwd(r["q"], r["k"], r["v"], off, b, e, True, scale)
    out, lse = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16), torch.from_numpy(l_ref).to("cuda:0").float()
    want = attn_bwd(r["q"], r["k"], r["v"], host_f64(out), r["do"], l_ref, off, b, e, True, scale)
    p = sp.make_params(dev["q"], dev["k"], out, off, b, e, True, scale)
    ws = torch.full((sp.slimpipe_attn_workspace_bytes(p, True),), 255, device="cuda:0", dtype=torch.uint8)
    assert sp.slimpipe_attn_call_path(p, True, -(-N // chunk) if chunk else 1, ws.numel()).small == 1
    res = []
    for add in (True, True, False):
        dk, dv = torch.full((B, N, H, D), 0.5, device="cuda:0"), torch.full((B, N, H, D), -0.25, device="cuda:0")
        kw = dict(dq_dtype=sp.F32, dkv_accumulate=add, workspace=ws)
        if chunk:
            cut = lambda x: [x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)]
            dkc, dvc = cut(dk), cut(dv)
            dq = sp.slimpipe_attn_bwd_chunked(dev["q"], cut(dev["k"]), cut(dev["v"]), out, dev["do"], lse, off, b, e, dkc, dvc, True, scale, **kw)
            dk, dv = torch.cat(dkc, 1), torch.cat(dvc, 1)
        else:
            dq = sp.slimpipe_attn_bwd(dev["q"], dev["k"], dev["v"], out, dev["do"], lse, off, b, e, dk, dv, True, scale, **kw)
        torch.cuda.synchronize()
        res.append((dq, dk, dv))
        inside = slice(b, e)
        for name, g, w, old in (("dq", dq, want[0], 0.0), ("dk", dk[:, inside], want[1][:, inside], 0.5), ("dv", dv[:, inside], want[2][:, inside], -0.25)):
            g = host_f64(g) - (old if add else 0.0)
            assert np.isfinite(g).all() and rel_l2(g, w) <= TOL_GRAD, name
        for x, old in ((dk, 0.5), (dv, -0.25)):
            assert (x[:, :b] == old).all() and (x[:, e:] == old).all(), "keys outside the range keep what they held"
    assert all(torch.equal(x, y) for x, y in zip(res[0], res[1])), "bit-reproducible"
