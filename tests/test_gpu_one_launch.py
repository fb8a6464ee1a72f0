"""Backward calls of fewer than two work items per compute unit run dq and dk/dv in one launch: the same items, so the same
bits as two launches (which the library makes while its per-kernel timing is on), at every workspace size."""
import math

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


# (batch, rows, keys, offset, q heads, kv heads, head_dim, chunk, causal, dq dtype, dq accumulate, dk/dv accumulate)
@pytest.mark.parametrize("B,s,N,off,Hq,Hkv,D,chunk,causal,dq,dqa,dkva", [
    (1, 512, 2048, 1536, 4, 4, 64, 0, True, "BF16", False, False),
    (1, 512, 512, 0, 4, 4, 64, 0, True, "BF16", False, True),
    (3, 337, 1238, 901, 12, 4, 64, 0, True, "F32", True, True),
    (1, 77, 9000, 8923, 8, 1, 128, 0, True, "BF16", False, True),
    (1, 300, 2560, 2200, 8, 2, 128, 512, True, "F32", False, False),
    (2, 40, 700, 3, 6, 2, 128, 0, False, "F32", True, False),
    (1, 1, 300, 299, 1, 1, 128, 0, True, "BF16", False, True)])
def test_one_launch_equals_two(B, s, N, off, Hq, Hkv, D, chunk, causal, dq, dqa, dkva):
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    mk = lambda n, h: torch.randn((B, n, h, D), device="cuda:0", generator=g).to(torch.bfloat16)
    q, do, k, v = mk(s, Hq), mk(s, Hq), mk(N, Hkv), mk(N, Hkv)
    split = (lambda x: [x[:, i:i + chunk].clone() for i in range(0, N, chunk)]) if chunk else (lambda x: x)
    fwd, bwd = (sp.slimpipe_attn_fwd_chunked, sp.slimpipe_attn_bwd_chunked) if chunk else (sp.slimpipe_attn_fwd, sp.slimpipe_attn_bwd)
    dqt = sp.F32 if dq == "F32" else sp.BF16
    for a, b in ((0, N), (130, N - 37)) if N > 300 else ((0, N), (0, 0)):
        o, l = fwd(q, split(k), split(v), off, a, b, causal, scale)
        need = sp.slimpipe_attn_workspace_bytes(sp.make_params(q, k, q, off, a, b, causal, scale), True)
        least = 2 * ((B * Hq * s * 4 + 255) // 256 * 256)
        base = None
        for nbytes in sorted({need, least, least + 256, (need + least) // 2 // 16 * 16}, reverse=True):
            say("one launch: %s keys [%d,%d) workspace %d" % ((B, s, N, off, Hq, Hkv, D, chunk, causal, dq, dqa, dkva), a, b, nbytes))
            res = []
            for two in (False, True):
                ws = torch.full((nbytes,), 0xff, device="cuda:0", dtype=torch.uint8)      # NaN patterns: nothing stale may be read
                dk, dv = split(torch.full((B, N, Hkv, D), 0.5, device="cuda:0")), split(torch.full((B, N, Hkv, D), 0.25, device="cuda:0"))
                out = torch.full((B, s, Hq, D), 0.125, device="cuda:0", dtype=torch.float32 if dq == "F32" else torch.bfloat16)
                sp.lib.slimpipe_attn_profile_enable(1 if two else 0)
                try:
                    bwd(q, split(k), split(v), o, do, l, off, a, b, dk, dv, causal, scale, dq=out, dq_dtype=dqt, dq_accumulate=dqa,
                        dkv_accumulate=dkva, workspace=ws)
                finally:
                    sp.lib.slimpipe_attn_profile_enable(0)
                torch.cuda.synchronize()
                if two:
                    sp.slimpipe_attn_profile_read()          # gives the events back
                res.append([out] + (dk + dv if chunk else [dk, dv]))
            for x, y in zip(*res):
                assert torch.equal(x, y)
                assert torch.isfinite(x.float()).all()
            if base is None:
                base = res[0]
            # other cuts only reorder float32 sums (each rounds to 2^-24 of the sum of magnitudes: a few hundred terms);
            # a bf16 dq may then round to the neighbouring value
            for x, y in zip(base, res[0]):
                d = (x.float() - y.float()).abs().max()
                assert float(d) <= (2.0 ** -7 if x.dtype == torch.bfloat16 else 1e-4) * max(1.0, float(x.float().abs().max())), nbytes
