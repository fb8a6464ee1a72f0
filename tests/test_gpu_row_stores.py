"""Output rows of the 256-row kernels, which leave through LDS as whole rows, and Q rows, which come in that way: ragged slices (waves
with some rows and with none), rows apart by odd multiples of 8 elements, both output types, dq added to what is there; nothing is
written between the rows."""
import math

import numpy as np
import pytest

from oracle import attn_fwd, attn_bwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, max_abs, rel_l2, out_err, TOL_OUT, TOL_LSE, TOL_GRAD

pytestmark = pytest.mark.gpu


def rows_apart(shape, dtype, pad, fill):
    """A [B, s, H, D] view whose rows are H * D + pad elements apart, and the buffer around it."""
    import torch
    B, s, H, D = shape
    wide = torch.full((B, s + 2, H * D + pad), fill, device="cuda:0", dtype=dtype)
    return wide[:, 1:1 + s, :H * D].unflatten(2, (H, D)), wide


def untouched(wide, s, width, fill):
    return bool((wide[:, 0] == fill).all() and (wide[:, s + 1:] == fill).all() and (wide[:, :, width:] == fill).all())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("s,Hq,Hkv,pad", [(1, 2, 1, 8), (33, 2, 2, 24), (257, 2, 1, 40), (300, 3, 1, 8)])
def test_rows_of_the_large_kernels(D, s, Hq, Hkv, pad):
    import torch
    import paper_2504_14519_amd as sp
    B, off = 2, 140
    N, scale = off + s, 1.0 / math.sqrt(D)
    say("rows of the large kernels: s=%d heads %d/%d D=%d, rows %d elements further apart" % (s, Hq, Hkv, D, pad))
    bits = {t: normal_bf16((B, N if t in "kv" else s, Hkv if t in "kv" else Hq, D), 71, t) for t in ("q", "k", "v", "do")}
    ref = {t: bf16_bits_to_f64(x) for t, x in bits.items()}
    o_ref, l_ref = attn_fwd(ref["q"], ref["k"], ref["v"], off, 0, N, True, scale)
    q, _ = rows_apart((B, s, Hq, D), torch.bfloat16, pad, 50.0)
    q.copy_(dev_bf16(bits["q"]))
    k, v, do = (dev_bf16(bits[t]) for t in ("k", "v", "do"))
    saved = None
    for code, dtype in ((sp.F32, torch.float32), (sp.BF16, torch.bfloat16)):
        out, wide = rows_apart((B, s, Hq, D), dtype, pad, 7.0)
        lse = torch.full((B, Hq, s), 7.0, device="cuda:0")
        sp.slimpipe_attn_fwd(q, k, v, off, 0, N, True, scale, out_dtype=code, out=out, lse=lse)      # (no workspace: 256-row blocks)
        torch.cuda.synchronize()
        eo, _ = out_err(host_f64(out), o_ref, code == sp.BF16)
        assert eo <= TOL_OUT and max_abs(host_f64(lse), l_ref) <= TOL_LSE
        assert untouched(wide, s, Hq * D, 7.0)
        saved = (out, lse)
    out, lse = saved
    dq_ref, _, _ = attn_bwd(ref["q"], ref["k"], ref["v"], host_f64(out), ref["do"], host_f64(lse), off, 0, N, True, scale)
    dk, dv = torch.zeros_like(k, dtype=torch.float32), torch.zeros_like(v, dtype=torch.float32)
    ws = torch.empty(2 * ((B * Hq * s * 4 + 255) // 256 * 256), device="cuda:0", dtype=torch.uint8)      # the statistics alone: no cuts
    for code, dtype, add in ((sp.BF16, torch.bfloat16, False), (sp.F32, torch.float32, False), (sp.F32, torch.float32, True)):
        dq, wide = rows_apart((B, s, Hq, D), dtype, pad, 7.0)
        start = torch.randn((B, s, Hq, D), generator=torch.Generator().manual_seed(3))
        dq.copy_(start)
        assert not sp.slimpipe_attn_call_path(sp.make_params(q, k, out, off, 0, N, True, scale), True, 1, ws.numel()).small
        sp.slimpipe_attn_bwd(q, k, v, out, do, lse, off, 0, N, dk, dv, True, scale, dq=dq, dq_dtype=code, dq_accumulate=add, workspace=ws)
        torch.cuda.synchronize()
        got = host_f64(dq) - (start.double().numpy() if add else 0.0)
        assert rel_l2(got, dq_ref) <= TOL_GRAD
        assert untouched(wide, s, Hq * D, 7.0)
