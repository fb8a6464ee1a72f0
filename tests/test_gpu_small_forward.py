"""Forward calls that take the 32-row kernel (few query blocks and a workspace, of the counters alone or with room for key ranges): against the fp64 oracle at the edges of its tiles and of the
sharing of keys among its eight waves, with and without key ranges, chunked keys, and rows without any key."""
import ctypes
import math

import numpy as np
import pytest

from oracle import attn_fwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, max_abs, out_err, TOL_OUT, TOL_LSE

pytestmark = pytest.mark.gpu


# B, rows, keys, query heads, kv heads, head_dim, q_offset, kv_begin, kv_end, causal, chunk rows, workspace
@pytest.mark.parametrize("B,s,N,Hq,Hkv,D,off,b,e,causal,chunk,ws", [
    (1, 1, 1, 1, 1, 128, 0, 0, 1, True, 0, True),
    (1, 31, 33, 2, 1, 128, 2, 0, 33, True, 0, True),             # two tiles: six waves without keys
    (2, 33, 257, 4, 2, 128, 224, 0, 257, True, 0, False),        # nine tiles of 32: the ninth goes to wave 0 again
    (1, 65, 513, 4, 4, 64, 448, 0, 513, True, 0, True),          # nine tiles of 64
    (1, 64, 700, 6, 2, 64, 0, 0, 700, False, 0, True),
    (1, 96, 1024, 4, 1, 128, 928, 130, 999, True, 256, True),    # range that begins and ends inside a tile, chunked
    (1, 96, 768, 4, 1, 64, 600, 70, 640, True, 256, False),
    (1, 40, 4096, 2, 1, 128, 4056, 0, 4096, True, 0, True),      # key ranges and a merge
    (1, 40, 3000, 2, 1, 64, 2960, 0, 3000, True, 0, True),
    (1, 100, 300, 2, 1, 128, 150, 200, 300, True, 0, True),      # the first 50 rows see no key of the range
    (1, 50, 300, 2, 1, 64, 150, 200, 300, True, 0, True),        # no row does
])
def test_small_forward(B, s, N, Hq, Hkv, D, off, b, e, causal, chunk, ws):
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    qb, kb, vb = (normal_bf16(shape, 32, t) for t, shape in (("q", (B, s, Hq, D)), ("k", (B, N, Hkv, D)), ("v", (B, N, Hkv, D))))
    q, k, v = (dev_bf16(x) for x in (qb, kb, vb))
    k[:, e:], v[:, e:] = float("nan"), float("nan")          # what the cache holds behind the range is not read
    wide = torch.full((B, s + 3, Hq, D), float("nan"), device="cuda:0", dtype=torch.bfloat16)       # a slice of a longer sequence
    wide[:, 2:2 + s] = q
    q = wide[:, 2:2 + s]
    o_ref, l_ref = attn_fwd(*(bf16_bits_to_f64(x) for x in (qb, kb, vb)), off, b, e, causal, scale)
    for dtype in (sp.BF16, sp.F32):
        out = torch.full((B, s, Hq, D), 7.0, device="cuda:0", dtype=torch.float32 if dtype == sp.F32 else torch.bfloat16)
        lse = torch.full((B, Hq, s), 7.0, device="cuda:0")
        p = sp.make_params(q, k, out, off, b, e, causal, scale, dtype)
        work = torch.full((sp.slimpipe_attn_workspace_bytes(p, False) if ws else 256,), 255, device="cuda:0", dtype=torch.uint8)
        path = sp.slimpipe_attn_call_path(p, False, 1, work.numel())
        assert path.small == (N > 1) and (path.ranges > 1) == (N >= 3000)          # (a single key: the 256-row blocks)
        say("small forward: B=%d s=%d N=%d %d/%d D=%d off=%d [%d,%d) causal %d chunk %d" % (B, s, N, Hq, Hkv, D, off, b, e, causal, chunk))
        if chunk:
            cut = lambda x: [x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)]
            sp.slimpipe_attn_fwd_chunked(q, cut(k), cut(v), off, b, e, causal, scale, out_dtype=dtype, out=out, lse=lse, workspace=work)
        else:
            sp.slimpipe_attn_fwd(q, k, v, off, b, e, causal, scale, out_dtype=dtype, out=out, lse=lse, workspace=work)
        torch.cuda.synchronize()
        eo, _ = out_err(host_f64(out), o_ref, dtype == sp.BF16)
        el = max_abs(host_f64(lse), l_ref)          # fails on a differing -inf pattern, too
        say("out max-abs %.3e lse %.3e" % (eo, el))
        assert eo <= TOL_OUT and el <= TOL_LSE


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("pad", [8, 16, 24, 40])
def test_small_forward_with_rows_apart(D, pad):
    """Row strides that are any multiple of 8 elements."""
    import torch
    import paper_2504_14519_amd as sp
    B, s, N, Hq, Hkv = 1, 70, 740, 8, 1
    scale = 1.0 / math.sqrt(D)

    def rows_apart(bits):
        x = dev_bf16(bits)
        wide = torch.full((x.shape[0], x.shape[1], x.shape[2] * D + pad), 100.0, device="cuda:0", dtype=x.dtype)
        view = wide[:, :, :x.shape[2] * D].unflatten(2, (x.shape[2], D))
        view.copy_(x)
        return view
    bits = [normal_bf16(shape, 35, t) for t, shape in (("q", (B, s, Hq, D)), ("k", (B, N, Hkv, D)), ("v", (B, N, Hkv, D)))]
    q, k, v = (rows_apart(x) for x in bits)
    o_ref, l_ref = attn_fwd(*(bf16_bits_to_f64(x) for x in bits), N - s, 0, N, True, scale)
    say("small forward, rows %d elements apart, D=%d" % (pad, D))
    p = sp.make_params(q, k, q, N - s, 0, N, True, scale, sp.F32)
    work = torch.full((sp.slimpipe_attn_workspace_bytes(p, False),), 255, device="cuda:0", dtype=torch.uint8)
    assert sp.slimpipe_attn_call_path(p, False, 1, work.numel()).small == 1
    out, lse = sp.slimpipe_attn_fwd(q, k, v, N - s, 0, N, True, scale, out_dtype=sp.F32, workspace=work)
    torch.cuda.synchronize()
    eo, _ = out_err(host_f64(out), o_ref, False)
    el = max_abs(host_f64(lse), l_ref)
    say("out max-abs %.3e lse %.3e" % (eo, el))
    assert eo <= TOL_OUT and el <= TOL_LSE
