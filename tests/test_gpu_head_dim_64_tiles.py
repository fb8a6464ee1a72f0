"""Backward at head_dim 64 against the fp64 oracle at the edges of its tiles (64 query rows of dk/dv, 128 keys of dq): rows and keys
one off a tile, a causal diagonal that starts inside one, a key range that begins and ends inside one, chunked keys."""
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
