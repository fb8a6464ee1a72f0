"""The merge for every count of parts (the kernel is compiled for 1, 2, 3, 4, 8 and 16 of them), both part types, empty parts
whose rows hold NaN, rows that are empty everywhere, against the same sums in float64."""
import math

import numpy as np
import pytest

from gpu_util import say, host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("f32", [True, False])
def test_merge_of_n_parts(n, f32):
    import torch
    import paper_2504_14519_amd as sp
    B, s, H, D = 2, 37, 3, 72          # (any head_dim that is a multiple of 8)
    say("merge of %d parts, float32 %s" % (n, f32))
    g = torch.Generator().manual_seed(7 + n)
    outs = [torch.randn((B, s, H, D), generator=g).to(torch.float32 if f32 else torch.bfloat16) for _ in range(n)]
    lses = [4.0 * torch.randn((B, H, s), generator=g) for _ in range(n)]
    for r in range(n):                 # part r sees nothing of every third row, no part sees anything of row 5
        empty = torch.zeros(s, dtype=torch.bool)
        empty[r % 3::3] = n > 1
        empty[5] = True
        lses[r][:, :, empty] = -math.inf
        outs[r][:, empty] = math.nan
    ld = np.stack([x.double().numpy() for x in lses])
    od = np.stack([host_f64(x) for x in outs])
    with np.errstate(all="ignore"):
        m = ld.max(0)
        e = np.where(np.isinf(ld), 0.0, np.exp(ld - np.where(np.isinf(m), 0.0, m)))
        tot = e.sum(0)
        lse_ref = np.where(tot > 0, m + np.log(tot), -np.inf)
        w = np.where(tot > 0, e / tot, 0.0).transpose(0, 1, 3, 2)[..., None]
    ref = np.where(w > 0, w * np.where(np.isnan(od), 0.0, od), 0.0).sum(0)
    out, lse = sp.slimpipe_attn_merge([x.to("cuda:0") for x in outs], [x.to("cuda:0") for x in lses], out_dtype=sp.F32)
    torch.cuda.synchronize()
    o, l = host_f64(out), host_f64(lse)
    assert np.array_equal(np.isinf(l), np.isinf(lse_ref)) and np.abs(np.where(np.isinf(l), 0, l - np.where(np.isinf(lse_ref), 0, lse_ref))).max() <= 1e-5
    # weights of exponents up to ~30 good to 30 * 2^-23 each, at most 16 terms of at most ~5
    assert np.isfinite(o).all() and np.abs(o - ref).max() <= 1e-4
    assert np.abs(o[:, 5]).max() == 0.0


@pytest.mark.parametrize("n", [1, 3, 6])
def test_rows_without_a_weight(n):
    """No part has a weight above zero: -inf in all, or not a number in some and -inf in the rest.  The row is 0, lse -inf."""
    import torch
    import paper_2504_14519_amd as sp
    B, s, H, D = 1, 70, 2, 64
    say("merge of %d parts without a weight" % n)
    outs = [torch.ones((B, s, H, D), device="cuda:0") for _ in range(n)]
    lses = [torch.full((B, H, s), -math.inf, device="cuda:0") for _ in range(n)]
    lses[0][:, :, 3:40] = math.nan
    lses[-1][:, :, 30:50] = math.nan
    out, lse = sp.slimpipe_attn_merge(outs, lses, out_dtype=sp.F32)
    torch.cuda.synchronize()
    assert (out == 0).all() and (lse == -math.inf).all()
