"""The forward's online softmax with a reference that has to move: scores that keep growing, jump, fall, or grow by little
from tile to tile, against the fp64 oracle through the C ABI."""
import math

import numpy as np
import pytest

from oracle import attn_fwd
from synth_inputs import normal_bf16, bf16_bits_to_f64
from gpu_util import say, dev_bf16, host_f64, max_abs, TOL_LSE

pytestmark = pytest.mark.gpu

S, N, HQ, HKV = 290, 1290, 4, 2
# factor on the keys (a power of two each, so that the scaled keys are bf16 again), by 128-key tile
RAMPS = {
    "growing": lambda t: 2.0 ** (t - 4),                       # the maximum moves in most tiles
    "jump and fall": lambda t: 64.0 if t == 5 else 1.0,        # one tile far above, the rest far below it
    "falling": lambda t: 2.0 ** (5 - t),
    "up and down by a little": lambda t: 2.0 if t % 2 else 0.5,
}


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("ramp", sorted(RAMPS))
def test_reference_follows_the_scores(D, ramp):
    import torch
    import paper_2504_14519_amd as sp
    scale = 1.0 / math.sqrt(D)
    f = np.array([RAMPS[ramp](j // 128) for j in range(N)]).reshape(1, N, 1, 1)
    q = bf16_bits_to_f64(normal_bf16((1, S, HQ, D), 17, "q"))
    k = bf16_bits_to_f64(normal_bf16((1, N, HKV, D), 17, "k")) * f
    v = bf16_bits_to_f64(normal_bf16((1, N, HKV, D), 17, "v"))
    dev = [torch.from_numpy(x).to(torch.float32).to(torch.bfloat16).to("cuda:0") for x in (q, k, v)]
    assert np.array_equal(host_f64(dev[1]), k), "the scaled keys are exact in bf16"
    for q_off, a, b in ((N - S, 0, N), (N - S, 130, N - 100), (0, 0, S)):
        say("softmax reference: D=%d, %s, keys [%d,%d) at %d" % (D, ramp, a, b, q_off))
        o, lse = sp.slimpipe_attn_fwd(dev[0], dev[1], dev[2], q_off, a, b, True, scale, out_dtype=sp.F32)
        torch.cuda.synchronize()
        o_ref, l_ref = attn_fwd(q, k, v, q_off, a, b, True, scale)
        # weights are rounded to bf16 (2^-9 each, and they sum to one); float32 scores of up to ~400 are good to 1e-3
        # of a nat at worst, which changes a weight by as much
        tol = (2.0 ** -9 + 1e-3) * np.abs(v).max()
        assert max_abs(host_f64(o), o_ref) <= tol
        assert max_abs(host_f64(lse), l_ref) <= TOL_LSE
