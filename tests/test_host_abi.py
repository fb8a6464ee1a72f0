"""CPU-only checks of the boundary: the shared library loads without a GPU, exports every function
the header declares, and its host-side validation returns the documented codes."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sp():
    import paper_2504_14519_amd as sp_
    return sp_


def declared_functions():
    """Every function declared in any header under include/."""
    names = set()
    inc = os.path.join(ROOT, "include")
    for f in sorted(os.listdir(inc)):
        if f.endswith(".h"):
            src = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, f)).read(), flags=re.S)
            names |= set(re.findall(r"\b(slimpipe_attn_[a-z0-9_]+)\s*\(", src))
    return sorted(names)


def test_library_exports_every_declared_symbol(sp):
    names = declared_functions()
    assert {"slimpipe_attn_fwd", "slimpipe_attn_bwd", "slimpipe_attn_merge", "slimpipe_attn_finalize_bf16",
            "slimpipe_attn_workspace_bytes", "slimpipe_attn_validate", "slimpipe_attn_strerror", "slimpipe_attn_init",
            "slimpipe_attn_profile_read", "slimpipe_attn_mfma_rate"} <= set(names)
    L = ctypes.CDLL(sp.library_path())
    for n in names:
        assert hasattr(L, n), n


def good_params(sp):
    p = sp.AttnParams()
    p.batch, p.s_q, p.n_q_heads, p.n_kv_heads, p.head_dim, p.causal = 1, 512, 8, 1, 128, 1
    p.kv_capacity, p.q_offset, p.kv_begin, p.kv_end = 4096, 1024, 0, 1536
    p.scale, p.out_dtype = 0.088, sp.BF16
    p.q_stride_b, p.q_stride_s, p.q_stride_h = 512 * 8 * 128, 8 * 128, 128
    p.kv_stride_b, p.kv_stride_s, p.kv_stride_h = 4096 * 128, 128, 128
    p.o_stride_b, p.o_stride_s, p.o_stride_h = 512 * 8 * 128, 8 * 128, 128
    p.do_stride_b, p.do_stride_s, p.do_stride_h = 512 * 8 * 128, 8 * 128, 128
    return p


def test_validation_codes(sp):
    assert sp.slimpipe_attn_validate(good_params(sp), True) == 0
    cases = [
        (dict(n_kv_heads=3), -2), (dict(head_dim=96), -2), (dict(s_q=0), -2), (dict(scale=0.0), -2),
        (dict(scale=float("nan")), -2), (dict(causal=2), -2), (dict(out_dtype=5), -2),
        (dict(kv_begin=2000, kv_end=1000), -3), (dict(kv_end=5000), -3), (dict(q_offset=-1), -3), (dict(kv_begin=-4), -3),
        (dict(q_stride_s=1023), -4), (dict(kv_stride_h=0), -4), (dict(o_stride_h=64), -4), (dict(do_stride_s=12), -4),
    ]
    for change, code in cases:
        p = good_params(sp)
        for k, v in change.items():
            setattr(p, k, v)
        assert sp.slimpipe_attn_validate(p, True) == code, (change, code)
    # d_out strides only matter to the backward
    p = good_params(sp)
    p.do_stride_s = 12
    assert sp.slimpipe_attn_validate(p, False) == 0
    # empty range is legal
    p = good_params(sp)
    p.kv_begin = p.kv_end = 700
    assert sp.slimpipe_attn_validate(p, True) == 0
    assert sp.lib.slimpipe_attn_validate(None, 0) == -1


def test_workspace_bytes_and_null_pointer_errors(sp):
    p = good_params(sp)
    assert sp.slimpipe_attn_workspace_bytes(p, False) == 256          # the ticket counter, no key ranges for this shape
    n = sp.slimpipe_attn_workspace_bytes(p, True)
    assert n >= 2 * 4 * 8 * 512 + 256 and n % 256 == 0
    # NULL data pointers are refused before anything touches the device
    rc = sp.lib.slimpipe_attn_fwd(ctypes.byref(p), None, None, None, None, None, None, 0, None)
    assert rc == -1
    rc = sp.lib.slimpipe_attn_finalize_bf16(None, None, 16, None)
    assert rc == -1
    assert "workspace" in sp.slimpipe_attn_strerror(-6)
    assert sp.slimpipe_attn_strerror(12345) == "unknown slimpipe status"


def test_equal_flop_cuts():
    from paper_2504_14519_amd.planner import equal_flop_cuts, visible_pairs_upto
    s, i = 4096, 20
    q_off = i * s
    for parts in (2, 3, 5):
        cuts = equal_flop_cuts(s, q_off, parts)
        assert cuts[0] == 0 and cuts[-1] == q_off + s and len(cuts) == parts + 1
        assert all(c % 128 == 0 for c in cuts) and cuts == sorted(cuts)
        total = visible_pairs_upto(s, q_off, q_off + s)
        work = [visible_pairs_upto(s, q_off, b) - visible_pairs_upto(s, q_off, a) for a, b in zip(cuts[:-1], cuts[1:])]
        assert sum(work) == total
        assert max(work) - min(work) <= 2 * 128 * s          # within an alignment step of equal
    # brute-force count of the closed form
    s, q_off = 7, 10
    for e in range(0, 20):
        brute = sum(1 for r in range(s) for j in range(e) if j <= q_off + r)
        assert visible_pairs_upto(s, q_off, e) == brute


def test_forward_workspace_asks_for_key_ranges_only_when_the_launch_is_small(sp):
    import types
    D = 128
    def params(s, Hq, Hkv, q_off, kv_end):
        q = types.SimpleNamespace(shape=(1, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
        k = types.SimpleNamespace(shape=(1, kv_end, Hkv, D), stride=lambda i, st=(kv_end * Hkv * D, Hkv * D, D, 1): st[i])
        return sp.make_params(q, k, q, q_off, 0, kv_end, True, None)
    per_range = lambda s, Hq: s * Hq * D * 4 + Hq * s * 4
    ticket = 256          # every forward workspace starts with the counter the workgroups take their items from
    # the benchmark shape: 64 query blocks x 8 heads = two full rounds on 256 compute units, nothing to gain
    assert sp.slimpipe_attn_workspace_bytes(params(16384, 8, 1, 15 * 16384, 16 * 16384), False) == ticket
    # 4096-row slices of the redistribution workload: 128 workgroups, two ranges fill the GPU
    assert sp.slimpipe_attn_workspace_bytes(params(4096, 8, 1, 31 * 4096, 32 * 4096), False) == ticket + 2 * per_range(4096, 8)
    # ... but never ranges shorter than 1024 keys
    assert sp.slimpipe_attn_workspace_bytes(params(256, 8, 1, 1024, 1280), False) == ticket
    assert sp.slimpipe_attn_workspace_bytes(params(256, 1, 1, 8192 - 256, 8192), False) == ticket + 8 * per_range(256, 1)
    # more ranges than 16 are refused, as are ranges outside the cache
    p = params(256, 8, 1, 1024, 1280)
    b, e = (ctypes.c_int64 * 17)(*([0] * 17)), (ctypes.c_int64 * 17)(*([64] * 17))
    one = (ctypes.c_void_p * 1)(64)
    args = lambda n: (ctypes.byref(p), 64, one, one, 1, 1280, n, b, e, 64, 64, None, None, None)
    assert sp.lib.slimpipe_attn_fwd_ranges(*args(17)) == -2
    assert sp.lib.slimpipe_attn_fwd_ranges(*args(0)) == -2
    e[3] = 1281
    assert sp.lib.slimpipe_attn_fwd_ranges(*args(4)) == -3


def test_backward_workspace_follows_the_split_policy(sp):
    """The backward workspace query = statistics + counters + partial dk/dv sums of the split the call would pick
    (+ partial dq of key ranges): the split policy of the dk/dv kernel, checked without a GPU (256 compute units are
    assumed when no device can be asked)."""
    import types
    D = 128
    def params(s, Hq, Hkv, q_off, kv_end):
        q = types.SimpleNamespace(shape=(1, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
        k = types.SimpleNamespace(shape=(1, kv_end, Hkv, D), stride=lambda i, st=(kv_end * Hkv * D, Hkv * D, D, 1): st[i])
        return sp.make_params(q, k, q, q_off, 0, kv_end, True, None)
    stats = lambda s, Hq: 2 * ((Hq * s * 4 + 255) // 256 * 256)
    counters = 256
    parts = lambda split, Hkv, keys: split * 2 * Hkv * keys * D * 4          # [chunk][dk, dv][kv head][keys][head_dim] floats
    dq_part = lambda s, Hq: s * Hq * D * 4
    # the benchmark workload, first slice: 64 key tiles for 256 compute units, streams of 4096 query tiles -> 8 chunks
    assert sp.slimpipe_attn_workspace_bytes(params(16384, 8, 1, 0, 16384), True) == stats(16384, 8) + counters + parts(8, 1, 16384)
    # its last slice: 1024 key tiles = 4 per compute unit -> 2 chunks bring them to 8
    assert sp.slimpipe_attn_workspace_bytes(params(16384, 8, 1, 15 * 16384, 16 * 16384), True) == stats(16384, 8) + counters + parts(2, 1, 16 * 16384)
    # the longest workload: 4096 key tiles, nothing to cut
    assert sp.slimpipe_attn_workspace_bytes(params(16384, 8, 1, 63 * 16384, 64 * 16384), True) == stats(16384, 8) + counters
    # 40 KV heads, 4096-row slices: 640 items of 128 query tiles (2.5 per compute unit): no split for whole rounds
    # once the counters are there; forward-like key ranges for dq (640 query blocks -> 2 ranges)
    assert sp.slimpipe_attn_workspace_bytes(params(4096, 40, 40, 0, 4096), True) == stats(4096, 40) + counters + 2 * dq_part(4096, 40)
    # the redistribution workload's last slice: 512 key tiles = 2 per compute unit, streams of 1024 tiles -> 2 chunks
    # (none below 512 tiles); dq in two key ranges
    assert sp.slimpipe_attn_workspace_bytes(params(4096, 8, 1, 31 * 4096, 32 * 4096), True) == \
        stats(4096, 8) + counters + parts(2, 1, 32 * 4096) + 2 * dq_part(4096, 8)


@pytest.mark.parametrize("s,Hq,Hkv,D,keys,batch", [(2387, 8, 1, 128, 52005, 1), (777, 8, 1, 128, 33777, 1), (512, 4, 4, 64, 2048, 1),
                                                  (300, 8, 2, 128, 2560, 1), (1337, 12, 4, 64, 4238, 3), (64, 8, 1, 128, 60000, 1)])
def test_backward_plan_is_made_for_the_workspace_it_gets(sp, s, Hq, Hkv, D, keys, batch):
    """A call of few items is cut for the room there is: whatever the workspace, the kind of item that takes longer AS CUT
    comes first in the launch (times of the items as the library states them), and the cuts fit."""
    import types
    q = types.SimpleNamespace(shape=(batch, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
    k = types.SimpleNamespace(shape=(batch, keys, Hkv, D), stride=lambda i, st=(keys * Hkv * D, Hkv * D, D, 1): st[i])
    p = sp.make_params(q, k, q, keys - s, 0, keys, True, None)
    stats = 2 * ((batch * Hq * s * 4 + 255) // 256 * 256)
    full = sp.slimpipe_attn_workspace_bytes(p, True)
    stream = (s + 31) // 32 * (Hq // Hkv)
    for room in sorted({stats, stats + 256, full} | {stats + 256 + (full - stats - 256) * i // 8 for i in range(1, 8)}):
        plan = sp.slimpipe_attn_bwd_plan(p, 1, room)
        assert plan.one_launch == 1
        assert plan.dq_items + plan.dkdv_items > 0
        dq = 8 + (2.4 if D == 128 else 1.4) * keys / 64 / plan.dq_ranges
        dkdv = 10 + (1.6 if D == 128 else 1.1) * stream / plan.dkdv_split
        assert plan.dq_first == (1 if dq > dkdv else 0), (room, plan.dkdv_split, plan.dq_ranges)
        parts = (plan.dkdv_split * 2 * batch * Hkv * ((keys + 255) // 256 * 256) * D * 4 if plan.dkdv_split > 1 else 0) + \
                (plan.dq_ranges * batch * s * Hq * D * 4 if plan.dq_ranges > 1 else 0)
        assert stats + (256 if room >= stats + 256 else 0) + parts <= room
        if room <= stats + 256:
            assert plan.dkdv_split == 1 and plan.dq_ranges == 1
    more = sp.slimpipe_attn_bwd_plan(p, 1, 4 * full)
    assert (more.dkdv_split, more.dq_ranges) == (plan.dkdv_split, plan.dq_ranges), "the query asks for all the room that is used"
    assert sp.lib.slimpipe_attn_bwd_plan(ctypes.byref(p), 1, stats - 16, ctypes.byref(more)) == -6


@pytest.mark.parametrize("s,Hq,Hkv,D,keys,batch,one", [(4096, 8, 1, 128, 57344, 1, 0), (8192, 8, 1, 128, 49152, 1, 0), (6000, 8, 1, 128, 60000, 1, 0),
                                                      (1608, 8, 1, 64, 22396, 2, 0), (3343, 8, 2, 128, 31065, 1, 1), (1989, 16, 16, 128, 2563, 1, 1)])
def test_backward_without_room_for_cuts_takes_the_faster_launches(sp, s, Hq, Hkv, D, keys, batch, one):
    """Long undivided items that one launch cannot even out run as two launches (measured: 3 to 8 % faster there); with the
    workspace the library asks for the same calls are cut and take one."""
    import types
    q = types.SimpleNamespace(shape=(batch, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
    k = types.SimpleNamespace(shape=(batch, keys, Hkv, D), stride=lambda i, st=(keys * Hkv * D, Hkv * D, D, 1): st[i])
    p = sp.make_params(q, k, q, keys - s, 0, keys, True, None)
    least = sp.slimpipe_attn_bwd_plan(p, 1, 2 * ((batch * Hq * s * 4 + 255) // 256 * 256) + 256)
    assert (least.one_launch, least.dkdv_split, least.dq_ranges) == (one, 1, 1)
    assert sp.slimpipe_attn_bwd_plan(p, 1, sp.slimpipe_attn_workspace_bytes(p, True)).one_launch == 1


def test_call_path_reports_the_kernels_of_a_call(sp):
    """The path query answers for the workspace it is asked about, and refuses what the calls refuse."""
    import types
    def params(B, s, Hq, Hkv, D, keys):
        q = types.SimpleNamespace(shape=(B, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
        k = types.SimpleNamespace(shape=(B, keys, Hkv, D), stride=lambda i, st=(keys * Hkv * D, Hkv * D, D, 1): st[i])
        return sp.make_params(q, k, q, keys - s, 0, keys, True, None)
    def path(p, bwd, room):
        c = sp.slimpipe_attn_call_path(p, bwd, 1, room)
        return (c.small, c.ranges, c.dq_tile_keys, c.dkdv_tile_rows) if bwd else (c.small, c.ranges)
    tiny, large = params(1, 512, 4, 4, 64, 2048), params(1, 16384, 8, 1, 128, 131072)
    assert [path(tiny, False, n) for n in (0, 256)] == [(0, 1), (1, 1)]
    least = 2 * 4 * 512 * 4
    assert path(tiny, True, sp.slimpipe_attn_workspace_bytes(tiny, True)) == (1, 1, 64, 32)
    assert path(tiny, True, least) == (0, 1, 64, 64)
    # above 32 dq items the model decides, not the number of items
    for s, small in ((256, 0), (257, 1), (288, 1), (480, 1), (511, 1)):
        p = params(1, s, 4, 4, 64, 2048)
        assert path(p, True, sp.slimpipe_attn_workspace_bytes(p, True))[0] == small, s
    assert path(large, False, 1 << 40) == (0, 1) and path(large, True, 1 << 40) == (0, 1, 64, 32)
    out = (ctypes.c_int32 * 4)()
    call = lambda p, bwd, n, room: sp.lib.slimpipe_attn_call_path(ctypes.byref(p), bwd, n, room, ctypes.cast(out, ctypes.POINTER(sp.binding.CallPath)))
    assert call(tiny, 1, 1, least - 16) == -6 and call(tiny, 0, 0, 0) == -2 and call(tiny, 0, 65, 0) == -2
    assert sp.lib.slimpipe_attn_call_path(ctypes.byref(tiny), 0, 1, 0, None) == -1 and sp.lib.slimpipe_attn_call_path(None, 0, 1, 0, None) == -1
    tiny.head_dim = 96
    assert call(tiny, 0, 1, 256) == -2


def test_forward_takes_the_small_kernel_only_with_the_workspace_it_asks_for(sp):
    """With a smaller workspace, or none, a forward call keeps the kernel of slimpipe_attn_fwd_ranges, undivided where no two ranges
    fit; with the one it asks for, or a larger one, it takes the same path."""
    import random
    import types
    rng = random.Random(4)
    shapes = [(1, 336, 8, 1, 64, 9624), (1, 1862, 8, 2, 64, 18838), (1, 1900, 4, 1, 128, 31226), (1, 512, 4, 1, 128, 8092), (1, 512, 4, 4, 64, 2048)]
    for _ in range(4000):
        Hq, Hkv = rng.choice([(8, 1), (4, 4), (8, 2), (12, 4), (16, 16), (4, 1), (40, 40), (1, 1)])
        s = int(2 ** rng.uniform(0, 13))
        shapes.append((rng.choice([1, 1, 2, 3]), s, Hq, Hkv, rng.choice([64, 128]), s + int(2 ** rng.uniform(0, 17))))
    asked_small = 0
    for B, s, Hq, Hkv, D, keys in shapes:
        q = types.SimpleNamespace(shape=(B, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
        k = types.SimpleNamespace(shape=(B, keys, Hkv, D), stride=lambda i, st=(keys * Hkv * D, Hkv * D, D, 1): st[i])
        p = sp.make_params(q, k, q, keys - s, 0, keys, True, None)
        need = sp.slimpipe_attn_workspace_bytes(p, False)
        path = lambda room: (lambda c: (c.small, c.ranges))(sp.slimpipe_attn_call_path(p, False, 1, room))
        per_range = lambda n: n * sum((x * 4 + 255) // 256 * 256 for x in (B * s * Hq * D, B * s * Hq))
        want = path(need)
        assert need == 256 + (per_range(want[1]) if want[1] > 1 else 0), (B, s, Hq, Hkv, D, keys)
        assert path(1 << 50) == want
        asked_small += want[0]
        for room in {0, 255, 256, need // 2, need - 16, 256 + per_range(2) - 16} - {need}:
            if room < need:
                small, ranges = path(room)
                assert small == 0 and (ranges == 1 or 256 + per_range(ranges) <= room), (B, s, Hq, Hkv, D, keys, room)
    assert 500 < asked_small < len(shapes) - 500


@pytest.mark.parametrize("B,s,Hq,Hkv,keys,dq_keys,dkdv_rows", [
    (4, 40, 40, 40, 5278, 64, 32), (8, 64, 32, 32, 870, 64, 32), (8, 160, 32, 8, 1184, 64, 32), (8, 512, 40, 40, 528, 64, 32),
    (8, 288, 16, 16, 800, 64, 32), (2, 1024, 16, 16, 13392, 128, 32), (2, 64, 32, 32, 16000, 128, 32),
    (4, 731, 12, 4, 8822, 128, 32), (4, 683, 64, 8, 1194, 64, 64), (4, 2432, 32, 32, 3921, 128, 64), (1, 8192, 16, 2, 40960, 128, 64)])
def test_two_launch_backward_of_head_dim_64_takes_large_tiles_where_walks_are_long(sp, B, s, Hq, Hkv, keys, dq_keys, dkdv_rows):
    """Measured: 64-row dk/dv tiles take up to 1.75 times as long on short or padded walks, 128-key dq tiles up to 1.2 times."""
    import types
    D = 64
    q = types.SimpleNamespace(shape=(B, s, Hq, D), stride=lambda i, st=(s * Hq * D, Hq * D, D, 1): st[i])
    k = types.SimpleNamespace(shape=(B, keys, Hkv, D), stride=lambda i, st=(keys * Hkv * D, Hkv * D, D, 1): st[i])
    p = sp.make_params(q, k, q, keys - s, 0, keys, True, None)
    need = sp.slimpipe_attn_workspace_bytes(p, True)
    assert sp.slimpipe_attn_bwd_plan(p, 1, need).one_launch == 0
    path = sp.slimpipe_attn_call_path(p, True, 1, need)
    assert (path.small, path.dq_tile_keys, path.dkdv_tile_rows) == (0, dq_keys, dkdv_rows)
