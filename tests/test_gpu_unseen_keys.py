"""What the cache holds at keys that no row sees is not read: before kv_begin and behind kv_end (inside a tile, on a chunk grid too), behind
the last position of a causal slice, in the gaps between the ranges of one launch.  Every call with NaN or infinities there returns, bit
for bit, what it returns with zeros, on every path: large and small forward, key ranges, one- and two-launch backward."""
import math

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


# B, rows, query heads, kv heads, keys, q_offset, kv_begin, kv_end, causal, chunk rows (0: one buffer), launches of the backward
@pytest.mark.parametrize("B,s,Hq,Hkv,N,off,b,e,causal,chunk,one", [
    (8, 200, 32, 32, 700, 400, 0, 320, False, 0, False),        # 64 keys past a 128-key tile
    (8, 200, 32, 32, 700, 300, 0, 501, True, 0, False),
    (8, 200, 32, 32, 768, 500, 70, 601, True, 256, False),      # begins and ends inside a tile of the chunk grid
    (8, 200, 32, 32, 768, 500, 193, 448, True, 256, False),
    (8, 200, 32, 32, 700, 100, 40, 700, True, 0, False),        # the slice ends before the range does
    (2, 300, 4, 2, 768, 500, 70, 601, True, 256, True),
    (2, 300, 4, 2, 768, 200, 333, 740, True, 256, True),        # the first rows see no key, the last keys are seen by no row
    (1, 512, 4, 4, 1000, 480, 0, 993, True, 0, True),
    (1, 40, 8, 1, 5000, 4700, 300, 4801, True, 0, True),
    (1, 40, 8, 1, 5000, 100, 300, 4801, True, 0, True),         # nothing is seen
    (1, 700, 8, 1, 9000, 2000, 100, 8000, True, 0, True),
])
@pytest.mark.parametrize("D", [64, 128])
def test_unseen_keys_are_not_read(B, s, Hq, Hkv, N, off, b, e, causal, chunk, one, D):
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    g = torch.Generator(device="cuda:0").manual_seed(11)
    mk = lambda n, h: torch.randn((B, n, h, D), device="cuda:0", generator=g).to(torch.bfloat16)
    q, do, k, v = mk(s, Hq), mk(s, Hq), mk(N, Hkv), mk(N, Hkv)
    seen_end = max(b, min(e, off + s)) if causal else e

    def with_unseen(fill):
        ks, vs = k.clone(), v.clone()
        for x in (ks, vs):
            x[:, :b], x[:, seen_end:] = fill, fill
        return ([x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)] for x in (ks, vs)) if chunk else (ks, vs)
    fwd, bwd = (sp.slimpipe_attn_fwd_chunked, sp.slimpipe_attn_bwd_chunked) if chunk else (sp.slimpipe_attn_fwd, sp.slimpipe_attn_bwd)
    p = sp.make_params(q, k, q, off, b, e, causal, scale)
    least = 2 * ((B * Hq * s * 4 + 255) // 256 * 256)
    third = (e - b) // 3
    ranges = [(b, b + third), (b + third + 7, b + 2 * third), (b + 2 * third + 30, e)]       # with gaps

    def run(fill):
        kk, vv = with_unseen(fill)
        res = []
        for ws in (None, torch.full((sp.slimpipe_attn_workspace_bytes(p, False),), 255, device="cuda:0", dtype=torch.uint8)):
            res += fwd(q, kk, vv, off, b, e, causal, scale, workspace=ws)
        o, l = res[0], res[1]
        for nbytes in (least, least + 256, sp.slimpipe_attn_workspace_bytes(p, True)):
            plan = sp.slimpipe_attn_bwd_plan(p, -(-N // chunk) if chunk else 1, nbytes)
            assert plan.one_launch == one
            dk, dv = torch.full((B, N, Hkv, D), 0.5, device="cuda:0"), torch.full((B, N, Hkv, D), 0.25, device="cuda:0")
            cut = (lambda x: [x[:, i:i + chunk].contiguous() for i in range(0, N, chunk)]) if chunk else (lambda x: x)
            dk, dv = cut(dk), cut(dv)
            ws = torch.full((nbytes,), 255, device="cuda:0", dtype=torch.uint8)
            res.append(bwd(q, kk, vv, o, do, l, off, b, e, dk, dv, causal, scale, dq_dtype=sp.F32, dkv_accumulate=False, workspace=ws))
            dk, dv = (torch.cat(x, 1) if chunk else x for x in (dk, dv))
            assert (dk[:, seen_end:e] == 0).all() and (dv[:, seen_end:e] == 0).all(), "gradients of keys that no row sees"
            res += [dk, dv]
        torch.cuda.synchronize()
        return res

    def run_ranges(fill):
        kk, vv = k.clone(), v.clone()
        for x in (kk, vv):
            edges = [0] + [i for r in ranges for i in r] + [N]
            for i in range(0, len(edges), 2):
                x[:, edges[i]:edges[i + 1]] = fill
            x[:, seen_end:] = fill
        res = sp.slimpipe_attn_fwd_ranges(q, kk, vv, off, ranges, causal, scale)
        torch.cuda.synchronize()
        return list(res)
    for name, call in (("call", run), ("ranges", run_ranges)):
        say("unseen keys, %s: D=%d B=%d s=%d %d/%d N=%d off=%d [%d,%d) causal %d chunk %d" % (name, D, B, s, Hq, Hkv, N, off, b, e, causal, chunk))
        want = call(0.0)
        assert all(not torch.isnan(x.float()).any() for x in want)
        for fill in (float("nan"), float("inf")):
            for i, (x, y) in enumerate(zip(want, call(fill))):
                assert torch.equal(x, y), (name, fill, i)
