"""Backward calls of fewer than two work items per compute unit run dq and dk/dv in one launch: the same items, so undivided the same
bits as in the two launches of a call of many sequences (at head_dim 64 where dk/dv walks tiles of the same rows, or has one
query head per K/V head: the order of the sums over a group is that of the tiles), and at every workspace size the same sums in another order."""
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
    stats = lambda batch: 2 * ((batch * Hq * s * 4 + 255) // 256 * 256)
    n_chunks = -(-N // chunk) if chunk else 1

    def backward(a, b, o, l, times, nbytes):
        """dq, dk, dv of the batch repeated `times` times, and whether the call is of one launch."""
        rep = lambda x: x.repeat(times, *[1] * (x.dim() - 1))
        ws = torch.full((nbytes,), 0xff, device="cuda:0", dtype=torch.uint8)      # NaN patterns: nothing stale may be read
        full = lambda x: torch.full((B * times, N, Hkv, D), x, device="cuda:0")
        dk, dv = split(full(0.5)), split(full(0.25))
        out = torch.full((B * times, s, Hq, D), 0.125, device="cuda:0", dtype=torch.float32 if dq == "F32" else torch.bfloat16)
        bwd(rep(q), split(rep(k)), split(rep(v)), rep(o), rep(do), rep(l), off, a, b, dk, dv, causal, scale, dq=out, dq_dtype=dqt,
            dq_accumulate=dqa, dkv_accumulate=dkva, workspace=ws)
        torch.cuda.synchronize()
        plan = sp.slimpipe_attn_bwd_plan(sp.make_params(rep(q), rep(k), rep(q), off, a, b, causal, scale), n_chunks, nbytes)
        return [out] + (dk + dv if chunk else [dk, dv]), plan

    for a, b in ((0, N), (130, N - 37)) if N > 300 else ((0, N), (0, 0)):
        o, l = fwd(q, split(k), split(v), off, a, b, causal, scale)
        need = sp.slimpipe_attn_workspace_bytes(sp.make_params(q, k, q, off, a, b, causal, scale), True)
        least = stats(B)
        say("one launch: %s keys [%d,%d) undivided" % ((B, s, N, off, Hq, Hkv, D, chunk, causal, dq, dqa, dkva), a, b))
        one, plan = backward(a, b, o, l, 1, least)
        assert plan.one_launch == (b > a) and plan.dkdv_split == 1 and plan.dq_ranges == 1
        times = -(-2 * plan.compute_units // plan.dkdv_items) if b > a else 2          # (key tiles alone are too many for one launch)
        two, plan = backward(a, b, o, l, times, stats(B * times))
        assert plan.one_launch == 0 and plan.dkdv_split == 1 and plan.dq_ranges == 1
        for x, y in zip(one, two):
            assert torch.isfinite(x.float()).all()
            for i in (0, times - 1):
                assert torch.equal(x, y[i * B:(i + 1) * B])
        for nbytes in sorted({need, max(need, least + 256), least + 256, (need + least) // 2 // 16 * 16} - {least}):
            say("one launch: workspace %d" % nbytes)
            cut, plan = backward(a, b, o, l, 1, nbytes)
            assert plan.one_launch == (b > a)
            # other cuts only reorder float32 sums (each rounds to 2^-24 of the sum of magnitudes: a few hundred terms);
            # a bf16 dq may then round to the neighbouring value
            for x, y in zip(one, cut):
                assert torch.isfinite(y.float()).all()
                d = (x.float() - y.float()).abs().max()
                assert float(d) <= (2.0 ** -7 if x.dtype == torch.bfloat16 else 1e-4) * max(1.0, float(x.float().abs().max())), nbytes


def test_timing_switch_times_the_launches_that_run():
    """The per-kernel times of the bench header are of the kernels a call runs without them."""
    import torch
    import paper_2504_14519_amd as sp
    s, N, H, D = 256, 1024, 4, 64
    mk = lambda n: torch.randn((1, n, H, D), device="cuda:0").to(torch.bfloat16)
    q, do, k, v = mk(s), mk(s), mk(N), mk(N)
    o, l = sp.slimpipe_attn_fwd(q, k, v, N - s, 0, N)
    say("timing switch: a small backward call")
    res = []
    for timing in (False, True):
        dk, dv = torch.zeros((1, N, H, D), device="cuda:0"), torch.zeros((1, N, H, D), device="cuda:0")
        sp.slimpipe_attn_profile_enable(timing)
        try:
            dq = sp.slimpipe_attn_bwd(q, k, v, o, do, l, N - s, 0, N, dk, dv)
        finally:
            sp.slimpipe_attn_profile_enable(False)
        torch.cuda.synchronize()
        res.append((dq, dk, dv))
        prof = sp.slimpipe_attn_profile_read()
    assert {kind: n for kind, (_, n) in prof.items() if n} == {"delta": 1, "bwd_both": 1, "both_reduce": 1}
    assert all(torch.equal(x, y) for x, y in zip(*res))
