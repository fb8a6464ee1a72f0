"""Backward at head_dim 64 against the fp64 oracle at the edges of its tiles (32 and 64 query rows of dk/dv, 64 and 128 keys of dq):
rows and keys one off a tile, a causal diagonal that starts inside one, a key range that begins and ends inside one, chunked
keys.  The first test's calls are short and take the smaller tiles, the second's name the tiles they take."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, rel_l2, TOL_GRAD

pytestmark = pytest.mark.gpu


# B, rows, keys, query heads, kv heads, q_offset, kv_begin, kv_end, chunk rows (0: one buffer)
@pytest.mark.parametrize("B,s,N,Hq,Hkv,off,b,e,chunk", [
    (1, 1, 129, 2, 2, 128, 0, 129, 0),
    (1, 63, 127, 2, 1, 64, 0, 127, 0),
    (1, 64, 128, 2, 1, 64, 0, 128, 0),
    (1, 65, 513, 4, 1, 448, 0, 513, 0),
    (2, 97, 385, 4, 2, 255, 70, 352, 0),
    (1, 200, 768, 6, 2, 500, 130, 700, 256),
    (12, 65, 321, 16, 16, 256, 0, 321, 0),        # enough items for a launch of each kind
])
def test_backward_head_dim_64(B, s, N, Hq, Hkv, off, b, e, chunk):
    import torch
    import paper_2504_14519_amd as sp
    D, scale = 64, 1.0 / math.sqrt(64)
    qb, kb, vb, dob = (normal_bf16(shape, 64, t) for t, shape in (("q", (B, s, Hq, D)), ("k", (B, N, Hkv, D)), ("v", (B, N, Hkv, D)), ("do", (B, s, Hq, D))))
    q64, k64, v64, do64 = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    q, k, v, do = (dev_bf16(x) for x in (qb, kb, vb, dob))
    o_ref, l_ref = attn_fwd(q64, k64, v64, off, b, e, True, scale)
    out = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16)
    lse = torch.from_numpy(l_ref).to("cuda:0").float()
    dq_r, dk_r, dv_r = attn_bwd(q64, k64, v64, host_f64(out), do64, l_ref, off, b, e, True, scale)
    dk, dv = torch.full((B, N, Hkv, D), 0.5, device="cuda:0"), torch.full((B, N, Hkv, D), -0.25, device="cuda:0")
    p = sp.make_params(q, k, out, off, b, e, True, scale)
    ws = torch.empty(sp.slimpipe_attn_workspace_bytes(p, True), device="cuda:0", dtype=torch.uint8)
    say("backward head_dim 64: B=%d s=%d N=%d %d/%d off=%d [%d,%d) chunk %d" % (B, s, N, Hq, Hkv, off, b, e, chunk))
    if chunk:
        cut = lambda x: [x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)]
        kc, vc, dkc, dvc = cut(k), cut(v), cut(dk), cut(dv)
        dq = sp.slimpipe_attn_bwd_chunked(q, kc, vc, out, do, lse, off, b, e, dkc, dvc, True, scale, dq_dtype=sp.F32, dkv_accumulate=True, workspace=ws)
        dk, dv = torch.cat(dkc, 1), torch.cat(dvc, 1)
    else:
        dq = sp.slimpipe_attn_bwd(q, k, v, out, do, lse, off, b, e, dk, dv, True, scale, dq_dtype=sp.F32, dkv_accumulate=True, workspace=ws)
    torch.cuda.synchronize()
    for name, g, r in (("dq", host_f64(dq), dq_r), ("dk", host_f64(dk) - 0.5, dk_r), ("dv", host_f64(dv) + 0.25, dv_r)):
        assert np.isfinite(g).all(), name
        err = rel_l2(g, r)
        say("%s rel-L2 %.3e" % (name, err))
        assert err <= TOL_GRAD, name
    outside = [i for i in range(N) if not b <= i < e]
    assert (dk[:, outside] == 0.5).all() and (dv[:, outside] == -0.25).all(), "keys outside the range keep what they held"


# rows, keys, query heads, kv heads, q_offset, kv_begin, kv_end, causal, chunk rows, copies of the sequence (enough items for the launches meant),
# workspace (what is asked for, 256 bytes less, or without room for cuts); one launch, chunks of the query stream, keys of a dq tile, rows of a dk/dv tile
@pytest.mark.parametrize("s,N,Hq,Hkv,off,b,e,causal,chunk,copies,room,one,split,dq_keys,dkdv_rows", [
    (639, 2300, 8, 2, 1661, 0, 2300, True, 0, 13, False, 0, 1, 128, 64),        # the last tile of either kind is short
    (639, 2304, 8, 2, 1500, 300, 2110, True, 256, 13, True, 0, 1, 128, 64),     # begins and ends inside a tile, chunked
    (1025, 2048, 8, 2, 900, 70, 1999, True, 512, 10, True, 0, 1, 128, 64),      # a single row in the last tile, keys that no row sees
    (64, 4352, 2, 2, 4136, 77, 4190, True, 256, 16, False, 0, 1, 128, 32),
    (250, 437, 64, 8, 187, 0, 437, True, 0, 8, True, 0, 1, 64, 64),
    (65, 321, 4, 4, 256, 0, 321, True, 0, 48, True, 0, 1, 64, 32),
    (703, 1280, 8, 2, 0, 33, 1200, False, 256, 13, True, 1, 1, 64, 64),
    (1023, 1500, 4, 2, 477, 0, 1500, True, 0, 1, False, 1, 1, 64, 64),
    (1023, 1500, 4, 2, 477, 0, 1500, True, 0, 7, True, 1, 3, 64, 64),           # chunks that begin inside a head
    (1535, 1792, 4, 2, 250, 70, 1700, True, 256, 6, True, 1, 4, 64, 64),
    (200, 768, 6, 2, 500, 130, 700, True, 256, 1, "less", 1, 4, 64, 32),
    (512, 2048, 4, 4, 1536, 0, 2048, True, 0, 1, "less", 1, 3, 64, 32),
    (400, 1500, 4, 1, 1100, 0, 1500, True, 0, 2, "less", 1, 6, 64, 32),
])
def test_backward_head_dim_64_tiles(s, N, Hq, Hkv, off, b, e, causal, chunk, copies, room, one, split, dq_keys, dkdv_rows):
    import torch
    import paper_2504_14519_amd as sp
    D, scale = 64, 1.0 / math.sqrt(64)
    qb, kb, vb, dob = (normal_bf16(shape, 65, t) for t, shape in (("q", (1, s, Hq, D)), ("k", (1, N, Hkv, D)), ("v", (1, N, Hkv, D)), ("do", (1, s, Hq, D))))
    q64, k64, v64, do64 = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    rep = lambda x: x.repeat(copies, 1, 1, 1)
    q, k, v, do = (rep(dev_bf16(x)) for x in (qb, kb, vb, dob))
    o_ref, l_ref = attn_fwd(q64, k64, v64, off, b, e, causal, scale)
    out = rep(torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16))
    lse = torch.from_numpy(l_ref).to("cuda:0").float().repeat(copies, 1, 1)
    ref = attn_bwd(q64, k64, v64, host_f64(out[:1]), do64, l_ref, off, b, e, causal, scale)
    p = sp.make_params(q, k, out, off, b, e, causal, scale)
    n_chunks = -(-N // chunk) if chunk else 1
    nbytes = sp.slimpipe_attn_workspace_bytes(p, True) - (256 if room == "less" else 0) if room else 2 * ((copies * Hq * s * 4 + 255) // 256 * 256) + 256
    plan, path = sp.slimpipe_attn_bwd_plan(p, n_chunks, nbytes), sp.slimpipe_attn_call_path(p, True, n_chunks, nbytes)
    assert (path.small, plan.one_launch, plan.dkdv_split, path.dq_tile_keys, path.dkdv_tile_rows) == (0, one, split, dq_keys, dkdv_rows)
    say("backward head_dim 64 tiles: s=%d N=%d %d/%d off=%d [%d,%d) causal %d chunk %d copies %d" % (s, N, Hq, Hkv, off, b, e, causal, chunk, copies))
    ws = torch.full((nbytes,), 255, device="cuda:0", dtype=torch.uint8)
    cut = (lambda x: [x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)]) if chunk else (lambda x: x)
    dk, dv = cut(torch.full((copies, N, Hkv, D), 0.5, device="cuda:0")), cut(torch.full((copies, N, Hkv, D), -0.25, device="cuda:0"))
    bwd = sp.slimpipe_attn_bwd_chunked if chunk else sp.slimpipe_attn_bwd
    dq = bwd(q, cut(k), cut(v), out, do, lse, off, b, e, dk, dv, causal, scale, dq_dtype=sp.F32, dkv_accumulate=True, workspace=ws)
    dk, dv = (torch.cat(x, 1) if chunk else x for x in (dk, dv))
    torch.cuda.synchronize()
    for name, g, r, old in (("dq", dq, ref[0], 0.0), ("dk", dk, ref[1], 0.5), ("dv", dv, ref[2], -0.25)):
        assert all(torch.equal(g[0], g[i]) for i in range(1, copies)), name
        x = host_f64(g[:1]) - old
        assert np.isfinite(x).all(), name
        err = rel_l2(x, r)
        say("%s rel-L2 %.3e" % (name, err))
        assert err <= TOL_GRAD, name
    outside = [i for i in range(N) if not b <= i < e]
    assert (dk[:, outside] == 0.5).all() and (dv[:, outside] == -0.25).all(), "keys outside the range keep what they held"
