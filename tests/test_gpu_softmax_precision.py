"""Precision of the forward's softmax on peaked scores.  The exponents of a row are taken relative to the largest score seen
so far, so a row's largest weight is exactly one and passes the rounding of the weights to bf16 unchanged."""
import math

import numpy as np
import pytest

from gpu_util import say, host_f64, max_abs

pytestmark = pytest.mark.gpu


def bf16(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to(torch.float32).to(torch.bfloat16)


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("ranges", [False, True])
def test_two_keys_share_a_row(D, ranges):
    """Every row sees two keys that matter, A with score 0 in the first tile and B above it in a later one; the others weigh
    less than 2^-40.  Each was the largest score when it came, so both weights are exactly one before float32 rescales the
    older one: nothing of the result has been rounded to bf16.  Errors left: the score in log2 units (up to 14, 2^-23
    relative, twice), two exponentials and a division in float32: below 14 * 2^-22 * ln 2 + 2^-20 < 2^-18 of the weights."""
    import torch
    import paper_2504_14519_amd as sp
    S, N, HQ, HKV = 160, 2100, 8, 4
    scale = 1.0 / math.sqrt(D)
    rng = np.random.default_rng(11)
    q, k = np.zeros((1, S, HQ, D)), np.zeros((1, N, HKV, D))
    # first component only: score (log2) = scale log2(e) u t with u = 1 .. 10.97 a bf16 number, t = sqrt(D) ln 2 on key B
    q[0, :, :, 0] = 1.0 + np.arange(S)[:, None] / 16.0 + np.arange(HQ)[None, :] / 256.0
    q = host_f64(bf16(q))
    k[0, :, :, 0] = -64.0 * math.sqrt(D)
    b_at = [130, 700, 1025, 2099]
    for h in range(HKV):
        k[0, 5, h, 0] = 0.0
        k[0, b_at[h], h, 0] = math.sqrt(D) * math.log(2.0)
    k = host_f64(bf16(k))
    v = host_f64(bf16(rng.standard_normal((1, N, HKV, D))))
    ws = None
    dq, dk, dv = [bf16(x).to("cuda:0") for x in (q, k, v)]
    if ranges:
        need = sp.slimpipe_attn_workspace_bytes(sp.make_params(dq, dk, dq, N, 0, N, True, scale, sp.F32), False)
        ws = torch.empty(need, device="cuda:0", dtype=torch.uint8)
    say("two keys a row: D=%d ranges=%s" % (D, ranges))
    o, lse = sp.slimpipe_attn_fwd(dq, dk, dv, N, 0, N, True, scale, out_dtype=sp.F32, workspace=ws)
    torch.cuda.synchronize()
    o, lse = host_f64(o), host_f64(lse)
    for h in range(HQ):
        hk = h // (HQ // HKV)
        x = scale * q[0, :, h, 0] * k[0, b_at[hk], hk, 0]          # nats
        wb = 1.0 / (1.0 + np.exp(-x))
        ref = (1.0 - wb)[:, None] * v[0, 5, hk] + wb[:, None] * v[0, b_at[hk], hk]
        assert np.abs(o[0, :, h] - ref).max() <= 2.0 ** -18 * np.abs(v[0, [5, b_at[hk]], hk]).max(), h
        assert np.abs(lse[0, h] - (x + np.log1p(np.exp(-x)))).max() <= 1e-5, h


@pytest.mark.parametrize("D,std", [(128, 1.0), (128, 4.0), (128, 8.0), (64, 4.0)])
def test_error_is_that_of_the_running_maximum(D, std):
    """Scores of the given standard deviation in nats.  The error of a float32 out against 64 bits may not exceed that of
    the same sums with weights rounded to bf16 relative to the running maximum of 128-key tiles, computed here in 64 bits, by
    more than a tenth: the two round the same weights (a float32 exponential moves a few of them across a rounding edge)."""
    import torch
    import paper_2504_14519_amd as sp
    S, N = 256, 8192
    scale = 1.0 / math.sqrt(D)
    rng = np.random.default_rng(5)
    q, k, v = [host_f64(bf16(f * rng.standard_normal((1, n, 1, D)))) for f, n in ((std, S), (1.0, N), (1.0, N))]
    say("peaked scores: D=%d std %g" % (D, std))
    o, lse = sp.slimpipe_attn_fwd(*[bf16(x).to("cuda:0") for x in (q, k, v)], N, 0, N, True, scale, out_dtype=sp.F32)
    torch.cuda.synchronize()
    s = scale * q[0, :, 0] @ k[0, :, 0].T
    ref_lse = np.log(np.exp(s - s.max(1, keepdims=True)).sum(1)) + s.max(1)
    ref = np.exp(s - ref_lse[:, None]) @ v[0, :, 0]
    m, l, acc = np.full(S, -np.inf), np.zeros(S), np.zeros((S, D))
    for t in range(0, N, 128):
        m_new = np.maximum(m, s[:, t:t + 128].max(1))
        p = np.exp(s[:, t:t + 128] - m_new[:, None])
        a = np.exp(m - m_new)
        l, acc, m = l * a + p.sum(1), acc * a[:, None] + host_f64(bf16(p)) @ v[0, t:t + 128, 0], m_new
    err = lambda x: np.linalg.norm(x - ref) / np.linalg.norm(ref)
    got, model = err(host_f64(o)[0, :, 0]), err(acc / l[:, None])
    say("out error %.3e, of the running maximum %.3e" % (got, model))
    assert got <= 1.1 * model
    assert max_abs(host_f64(lse)[0, 0], ref_lse) <= 1e-4
