"""Backward calls that take the kernel of 32-row and 32-key items (few work items and the workspace the library asks for): against
the fp64 oracle at the edges of its tiles, of the sharing among its eight waves and of a causal diagonal, chunked keys, a range
that begins and ends inside a tile, rows without any key; twice, bit for bit."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, rel_l2, TOL_GRAD

pytestmark = pytest.mark.gpu


# B, rows, keys, query heads, kv heads, head_dim, q_offset, kv_begin, kv_end, causal, chunk rows
@pytest.mark.parametrize("B,s,N,Hq,Hkv,D,off,b,e,causal,chunk", [
    (1, 257, 513, 8, 4, 128, 256, 0, 513, True, 0),        # 18 query tiles of a group, 17 key tiles
    (2, 256, 1024, 4, 4, 64, 768, 0, 1024, True, 0),
    (2, 161, 545, 6, 2, 64, 384, 0, 545, True, 0),
    (1, 300, 900, 8, 1, 128, 500, 37, 777, True, 0),
    (1, 190, 1024, 12, 2, 128, 800, 300, 985, True, 256),
    (3, 190, 1024, 4, 1, 64, 800, 300, 985, True, 256),
    (1, 129, 600, 16, 2, 64, 0, 0, 600, False, 0),
    (1, 400, 700, 8, 1, 128, 150, 300, 700, True, 0),      # the first 150 rows see no key of the range
    (1, 480, 2048, 4, 4, 64, 1568, 0, 2048, True, 0),      # 60, 33 and 36 dq items
    (3, 321, 700, 1, 1, 128, 379, 0, 700, True, 0),
    (2, 43, 768, 9, 3, 64, 700, 100, 743, True, 256),
])
def test_small_backward(B, s, N, Hq, Hkv, D, off, b, e, causal, chunk):
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    qb, kb, vb, dob = (normal_bf16(shape, 33, t) for t, shape in (("q", (B, s, Hq, D)), ("k", (B, N, Hkv, D)), ("v", (B, N, Hkv, D)), ("do", (B, s, Hq, D))))
    q64, k64, v64, do64 = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    q, k, v, do = (dev_bf16(x) for x in (qb, kb, vb, dob))
    k[:, e:], v[:, e:] = float("nan"), float("nan")          # what the cache holds behind the range is not read

    def inside_of_longer(x, fill):                         # a slice of a longer sequence
        wide = torch.full((B, s + 3, Hq, D), fill, device="cuda:0", dtype=x.dtype)
        wide[:, 2:2 + s] = x
        return wide[:, 2:2 + s]
    q, do = inside_of_longer(q, float("nan")), inside_of_longer(do, float("nan"))
    o_ref, l_ref = attn_fwd(q64, k64, v64, off, b, e, causal, scale)
    out = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16)
    lse = torch.from_numpy(l_ref).to("cuda:0").float()
    dq_r, dk_r, dv_r = attn_bwd(q64, k64, v64, host_f64(out), do64, l_ref, off, b, e, causal, scale)
    p = sp.make_params(q, k, out, off, b, e, causal, scale)
    assert sp.slimpipe_attn_call_path(p, True, -(-N // chunk) if chunk else 1, sp.slimpipe_attn_workspace_bytes(p, True)).small == 1
    res = []
    for dtype, accumulate in ((sp.F32, True), (sp.F32, True), (sp.BF16, False)):
        say("small backward: B=%d s=%d N=%d %d/%d D=%d off=%d [%d,%d) causal %d chunk %d" % (B, s, N, Hq, Hkv, D, off, b, e, causal, chunk))
        ws = torch.full((sp.slimpipe_attn_workspace_bytes(p, True),), 255, device="cuda:0", dtype=torch.uint8)
        dk, dv = torch.full((B, N, Hkv, D), 0.5, device="cuda:0"), torch.full((B, N, Hkv, D), -0.25, device="cuda:0")
        dq = inside_of_longer(torch.full((B, s, Hq, D), 2.0, device="cuda:0", dtype=torch.float32 if dtype == sp.F32 else torch.bfloat16), 9.0)
        kw = dict(dq=dq, dq_dtype=dtype, dq_accumulate=accumulate, dkv_accumulate=accumulate, workspace=ws)
        if chunk:
            cut = lambda x: [x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)]
            dkc, dvc = cut(dk), cut(dv)
            sp.slimpipe_attn_bwd_chunked(q, cut(k), cut(v), out, do, lse, off, b, e, dkc, dvc, causal, scale, **kw)
            dk, dv = torch.cat(dkc, 1), torch.cat(dvc, 1)
        else:
            sp.slimpipe_attn_bwd(q, k, v, out, do, lse, off, b, e, dk, dv, causal, scale, **kw)
        torch.cuda.synchronize()
        assert (dq._base[:, :2] == 9.0).all() and (dq._base[:, 2 + s:] == 9.0).all(), "rows beside the slice keep what they held"
        inside = [i for i in range(N) if b <= i < e]
        outside = [i for i in range(N) if not b <= i < e]
        old = (2.0, 0.5, -0.25) if accumulate else (0.0, 0.0, 0.0)
        for name, g, r, o in (("dq", host_f64(dq), dq_r, old[0]), ("dk", host_f64(dk)[:, inside], dk_r[:, inside], old[1]),
                              ("dv", host_f64(dv)[:, inside], dv_r[:, inside], old[2])):
            assert np.isfinite(g).all(), name
            err = rel_l2(g - o, r)
            say("%s rel-L2 %.3e" % (name, err))
            assert err <= TOL_GRAD, name
        assert (dk[:, outside] == 0.5).all() and (dv[:, outside] == -0.25).all(), "keys outside the range keep what they held"
        res.append((dq, dk, dv))
    assert all(torch.equal(x, y) for x, y in zip(res[0], res[1]))


def _rows_apart(x, pad, fill):
    """x with `pad` more elements between its rows, which hold `fill`."""
    import torch
    B, n, H, D = x.shape
    wide = torch.full((B, n, H * D + pad), fill, device=x.device, dtype=x.dtype)
    view = wide[:, :, :H * D].unflatten(2, (H, D))
    view.copy_(x)
    return view


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("pad", [8, 16, 24, 40])
def test_small_backward_with_rows_apart(D, pad):
    """Row strides that are any multiple of 8 elements: the bytes between the rows are not read, and not written."""
    import torch
    import paper_2504_14519_amd as sp
    B, s, N, Hq, Hkv = 1, 300, 740, 8, 1
    off, scale = N - s, 1.0 / math.sqrt(D)
    qb, kb, vb, dob = (normal_bf16(shape, 34, t) for t, shape in (("q", (B, s, Hq, D)), ("k", (B, N, Hkv, D)), ("v", (B, N, Hkv, D)), ("do", (B, s, Hq, D))))
    q64, k64, v64, do64 = (bf16_bits_to_f64(x) for x in (qb, kb, vb, dob))
    q, k, v, do = (_rows_apart(dev_bf16(x), pad, 100.0) for x in (qb, kb, vb, dob))
    o_ref, l_ref = attn_fwd(q64, k64, v64, off, 0, N, True, scale)
    out = torch.from_numpy(o_ref).to("cuda:0").to(torch.bfloat16)
    lse = torch.from_numpy(l_ref).to("cuda:0").float()
    ref = attn_bwd(q64, k64, v64, host_f64(out), do64, l_ref, off, 0, N, True, scale)
    say("small backward, rows %d elements apart, D=%d" % (pad, D))
    dk, dv = (_rows_apart(torch.zeros((B, N, Hkv, D), device="cuda:0"), pad, 5.0) for _ in range(2))
    dq = _rows_apart(torch.zeros((B, s, Hq, D), device="cuda:0"), pad, 5.0)
    p = sp.make_params(q, k, out, off, 0, N, True, scale)
    ws = torch.empty(sp.slimpipe_attn_workspace_bytes(p, True), device="cuda:0", dtype=torch.uint8)
    assert sp.slimpipe_attn_call_path(p, True, 1, ws.numel()).small == 1
    sp.slimpipe_attn_bwd(q, k, v, out, do, lse, off, 0, N, dk, dv, True, scale, dq=dq, dq_dtype=sp.F32, dkv_accumulate=False, workspace=ws)
    torch.cuda.synchronize()
    for name, g, r in zip(("dq", "dk", "dv"), (dq, dk, dv), ref):
        err = rel_l2(host_f64(g), r)
        say("%s rel-L2 %.3e" % (name, err))
        assert err <= TOL_GRAD, name
        assert (g._base[:, :, -pad:] == 5.0).all(), name
