"""How the kernel of 32-row and 32-key items would do a backward call: what the query reports (host code only)."""
import ctypes
import types

import pytest


@pytest.fixture(scope="module")
def sp():
    import paper_2504_14519_amd as sp_
    return sp_


def params(sp, B, s, N, Hq, Hkv, D=64, causal=True, off=None, b=0, e=None):
    q = types.SimpleNamespace(shape=(B, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
    k = types.SimpleNamespace(shape=(B, N, Hkv, D), stride=lambda i, st=(N * Hkv * D, Hkv * D, D, 1): st[i])
    return sp.make_params(q, k, q, N - s if off is None else off, b, N if e is None else e, causal, None)


def way(sp, p, n_chunks=1, room=None):
    m = sp.slimpipe_attn_small_bwd_plan(p, n_chunks, sp.slimpipe_attn_workspace_bytes(p, True) if room is None else room)
    return m.small, m.key_blocks, m.own_statistics


@pytest.mark.parametrize("B,s,N,Hq,Hkv,causal,blocks,own", [
    (1, 512, 2048, 4, 4, True, 2, 1),
    (1, 300, 700, 4, 4, True, 1, 1),
    (1, 192, 500, 8, 1, True, 1, 1),           # 6 steps of a wave, every item on a unit of its own
    (1, 193, 500, 8, 1, True, 1, 0),
    (1, 618, 3090, 12, 4, True, 2, 0),
    # measured with one block / two: 19.5 / 25.6, 20.4 / 23.6, 14.2 / 17.6, 19.8 / 22.6 us
    (1, 1920, 2679, 2, 2, True, 1, 0),
    (1, 1632, 1644, 4, 4, True, 1, 1),
    (2, 1024, 1061, 2, 2, True, 1, 1),
    (1, 1536, 1613, 4, 4, True, 1, 1),
    # measured behind a delta kernel / without: 54.9 / 64.8, 33.6 / 37.5 us
    (1, 1334, 12925, 2, 2, False, None, 0),
    (1, 378, 3621, 12, 4, True, None, 0),
])
def test_two_blocks_and_own_statistics_where_they_are_faster(sp, B, s, N, Hq, Hkv, causal, blocks, own):
    small, b, o = way(sp, params(sp, B, s, N, Hq, Hkv, causal=causal))
    assert small == 1 and o == own and b in ((1, 2) if blocks is None else (blocks,))


@pytest.mark.parametrize("s,N,off,b,e,chunk", [
    (512, 2048, 1536, 0, 2048, 0), (500, 2010, 1510, 0, 2010, 0), (300, 2600, 2200, 37, 2500, 0), (300, 2560, 2200, 37, 2500, 256),
    (600, 2048, 1500, 0, 2048, 0), (512, 2048, 1400, 0, 2048, 0)])
def test_calls_of_two_key_blocks_take_two(sp, s, N, off, b, e, chunk):
    assert way(sp, params(sp, 1, s, N, 4, 4, off=off, b=b, e=e), -(-N // chunk) if chunk else 1) == (1, 2, 1)


def test_query_of_other_calls(sp):
    small, large, d128 = params(sp, 1, 512, 2048, 4, 4), params(sp, 1, 16384, 131072, 8, 1, D=128), params(sp, 1, 257, 513, 8, 4, D=128)
    least = 2 * 4 * 512 * 4
    assert way(sp, small, room=least) == (0, 0, 0) and way(sp, large) == (0, 0, 0)
    assert way(sp, d128) == (1, 1, 0)
    out = sp.binding.SmallBwdPlan()
    call = lambda p, n, room, to: sp.lib.slimpipe_attn_small_bwd_plan(ctypes.byref(p) if p else None, n, room, ctypes.byref(to) if to else None)
    assert call(None, 1, 0, out) == -1 and call(small, 1, 1 << 30, None) == -1
    assert call(small, 0, 1 << 30, out) == -2 and call(small, 65, 1 << 30, out) == -2 and call(small, 1, least - 16, out) == -6
    small.head_dim = 96
    assert call(small, 1, 1 << 30, out) == -2
