"""ctypes binding of libslimpipe_attn.so: argument marshalling only.

Same entry-point names as the C header.  Tensors are torch tensors on the GPU; torch supplies
device memory and the current stream, every step of the computation runs in the library's kernels.
There is no fallback: if the shared library is missing the import fails.
"""
import ctypes
import math
import os

# torch before the library: the tensors and streams handed to the library come from torch's HIP runtime, so that runtime has
# to be the one already in the process when the library's dependency on libamdhip64 is resolved (loaded the other
# way round, the library can end up on a second runtime instance that sees no device)
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libslimpipe_attn.so")

BF16, F32 = 0, 1


class SlimpipeError(RuntimeError):
    pass


class AttnParams(ctypes.Structure):
    _fields_ = [
        ("batch", ctypes.c_int32), ("s_q", ctypes.c_int32), ("n_q_heads", ctypes.c_int32),
        ("n_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32), ("causal", ctypes.c_int32),
        ("kv_capacity", ctypes.c_int64), ("q_offset", ctypes.c_int64), ("kv_begin", ctypes.c_int64),
        ("kv_end", ctypes.c_int64), ("scale", ctypes.c_float), ("out_dtype", ctypes.c_int32),
        ("q_stride_b", ctypes.c_int64), ("q_stride_s", ctypes.c_int64), ("q_stride_h", ctypes.c_int64),
        ("kv_stride_b", ctypes.c_int64), ("kv_stride_s", ctypes.c_int64), ("kv_stride_h", ctypes.c_int64),
        ("o_stride_b", ctypes.c_int64), ("o_stride_s", ctypes.c_int64), ("o_stride_h", ctypes.c_int64),
        ("do_stride_b", ctypes.c_int64), ("do_stride_s", ctypes.c_int64), ("do_stride_h", ctypes.c_int64),
    ]


class BwdPlan(ctypes.Structure):
    _fields_ = [
        ("one_launch", ctypes.c_int32), ("dq_first", ctypes.c_int32), ("dkdv_split", ctypes.c_int32), ("dq_ranges", ctypes.c_int32),
        ("dkdv_items", ctypes.c_int64), ("dq_items", ctypes.c_int64), ("compute_units", ctypes.c_int32), ("dq_by_xcd", ctypes.c_int32),
    ]


class CallPath(ctypes.Structure):
    _fields_ = [("small", ctypes.c_int32), ("ranges", ctypes.c_int32), ("dq_tile_keys", ctypes.c_int32), ("dkdv_tile_rows", ctypes.c_int32)]


class SmallBwdPlan(ctypes.Structure):
    _fields_ = [("small", ctypes.c_int32), ("key_blocks", ctypes.c_int32), ("own_statistics", ctypes.c_int32), ("dq_first", ctypes.c_int32)]


def library_path():
    return _LIB_PATH


def _load():
    if not os.path.exists(_LIB_PATH):
        # nothing built yet: compile the HIP library now (hipcc cross-compiles without a GPU).  There is no
        # fallback path: if that fails, so does the import.
        try:
            from .build import build as _build
            _build()
        except Exception as e:
            raise ImportError("libslimpipe_attn.so is not built and building it failed (%s): run "
                              "`python paper_2504_14519_amd/build.py`" % e)
    L = ctypes.CDLL(_LIB_PATH)
    P = ctypes.POINTER(AttnParams)
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    L.slimpipe_attn_init.argtypes = []
    L.slimpipe_attn_init.restype = ctypes.c_int
    L.slimpipe_attn_validate.argtypes = [P, ctypes.c_int]
    L.slimpipe_attn_validate.restype = ctypes.c_int
    L.slimpipe_attn_workspace_bytes.argtypes = [P, ctypes.c_int, ctypes.POINTER(ctypes.c_size_t)]
    L.slimpipe_attn_workspace_bytes.restype = ctypes.c_int
    L.slimpipe_attn_fwd.argtypes = [P, vp, vp, vp, vp, vp, vp, ctypes.c_size_t, vp]
    L.slimpipe_attn_fwd.restype = ctypes.c_int
    L.slimpipe_attn_bwd.argtypes = [P, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp, vp, i32, vp, ctypes.c_size_t, vp]
    L.slimpipe_attn_bwd.restype = ctypes.c_int
    L.slimpipe_attn_bwd_noalloc.argtypes = [P, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp, vp, i32, vp]
    L.slimpipe_attn_bwd_noalloc.restype = ctypes.c_int
    L.slimpipe_attn_noalloc_max_rows.argtypes = []
    L.slimpipe_attn_noalloc_max_rows.restype = ctypes.c_int
    pp = ctypes.POINTER(vp)
    L.slimpipe_attn_fwd_chunked.argtypes = [P, vp, pp, pp, i32, i64, vp, vp, vp, ctypes.c_size_t, vp]
    L.slimpipe_attn_fwd_chunked.restype = ctypes.c_int
    L.slimpipe_attn_bwd_chunked.argtypes = [P, vp, pp, pp, i32, i64, vp, vp, vp, vp, i32, i32, pp, pp, i32, vp, ctypes.c_size_t, vp]
    L.slimpipe_attn_bwd_chunked.restype = ctypes.c_int
    L.slimpipe_attn_fwd_ranges.argtypes = [P, vp, pp, pp, i32, i64, i32, ctypes.POINTER(i64), ctypes.POINTER(i64), vp, vp, vp, vp, vp]
    L.slimpipe_attn_fwd_ranges.restype = ctypes.c_int
    L.slimpipe_attn_merge.argtypes = [i32, ctypes.POINTER(vp), ctypes.POINTER(vp), i32, i32, i32, i32, i32, vp, i32, vp, vp]
    L.slimpipe_attn_merge.restype = ctypes.c_int
    L.slimpipe_attn_finalize_bf16.argtypes = [vp, vp, i64, vp]
    L.slimpipe_attn_finalize_bf16.restype = ctypes.c_int
    L.slimpipe_attn_mfma_rate.argtypes = [ctypes.c_int, vp, ctypes.POINTER(ctypes.c_double), vp]
    L.slimpipe_attn_mfma_rate.restype = ctypes.c_int
    L.slimpipe_attn_dq_atomic_probe.argtypes = [vp, i32, i32, i32, i32, i32, i32, i32, i32, vp, ctypes.POINTER(ctypes.c_double), vp]
    L.slimpipe_attn_dq_atomic_probe.restype = ctypes.c_int
    L.slimpipe_attn_xcd_rate.argtypes = [i32, i32, vp, vp, vp, vp]
    L.slimpipe_attn_xcd_rate.restype = ctypes.c_int
    L.slimpipe_attn_profile_enable.argtypes = [ctypes.c_int]
    L.slimpipe_attn_profile_enable.restype = ctypes.c_int
    L.slimpipe_attn_profile_read.argtypes = [ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int64)]
    L.slimpipe_attn_profile_read.restype = ctypes.c_int
    L.slimpipe_attn_bwd_plan.argtypes = [P, i32, ctypes.c_size_t, ctypes.POINTER(BwdPlan)]
    L.slimpipe_attn_bwd_plan.restype = ctypes.c_int
    L.slimpipe_attn_call_path.argtypes = [P, ctypes.c_int, i32, ctypes.c_size_t, ctypes.POINTER(CallPath)]
    L.slimpipe_attn_call_path.restype = ctypes.c_int
    L.slimpipe_attn_small_bwd_plan.argtypes = [P, i32, ctypes.c_size_t, ctypes.POINTER(SmallBwdPlan)]
    L.slimpipe_attn_small_bwd_plan.restype = ctypes.c_int
    L.slimpipe_attn_strerror.argtypes = [ctypes.c_int]
    L.slimpipe_attn_strerror.restype = ctypes.c_char_p
    return L


lib = _load()


def slimpipe_attn_strerror(code):
    return lib.slimpipe_attn_strerror(int(code)).decode()


def _check(rc, what):
    if rc != 0:
        raise SlimpipeError("%s failed: %d (%s)" % (what, rc, slimpipe_attn_strerror(rc)))


def _stream():
    # the raw handle of the current device's current stream, through two private functions of torch: 0.3 us; the public call
    # builds a stream object, 2.9 us
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


def _same_strides(a, b):
    """Equal shapes and equal strides on every dimension longer than one."""
    if a.stride() == b.stride() and a.shape == b.shape:
        return True
    return a.shape == b.shape and all(sa == sb for n, sa, sb in zip(a.shape, a.stride(), b.stride()) if n > 1)


def _params(q, k, out_like, d_out, q_offset, kv_begin, kv_end, causal, scale, out_dtype):
    # strides as whole tuples: a question to a tensor is 0.1 us, and every call fills one of these (2.3 -> 1.3 us)
    B, s, Hq, D = q.shape
    k_shape, sq, sk, so, sd = k.shape, q.stride(), k.stride(), out_like.stride(), d_out.stride()
    # in the order of AttnParams
    return AttnParams(B, s, Hq, k_shape[2], D, 1 if causal else 0, k_shape[1], q_offset, kv_begin, kv_end,
                      float(scale) if scale is not None else 1.0 / math.sqrt(D), out_dtype, sq[0], sq[1], sq[2],
                      sk[0], sk[1], sk[2], so[0], so[1], so[2], sd[0], sd[1], sd[2])


class _Layout:
    """Shape and strides of anything that has a shape and answers stride(i)."""
    def __init__(self, x):
        self.shape = x.shape
        self._strides = x.stride(0), x.stride(1), x.stride(2)

    def stride(self):
        return self._strides


def make_params(q, k, out_like, q_offset, kv_begin, kv_end, causal, scale, out_dtype=BF16):
    """Fill the parameter block from shapes/strides.  q [B,s,Hq,D], k [B,Nkv,Hkv,D]; the strides of d_out are those of out."""
    out_like = _Layout(out_like)
    return _params(_Layout(q), _Layout(k), out_like, out_like, q_offset, kv_begin, kv_end, causal, scale, out_dtype)


def slimpipe_attn_init():
    """Prepare the current device for launches (needed once per device before a HIP graph capture)."""
    _check(lib.slimpipe_attn_init(), "slimpipe_attn_init")


def slimpipe_attn_validate(params, is_bwd=False):
    return lib.slimpipe_attn_validate(ctypes.byref(params), 1 if is_bwd else 0)


def slimpipe_attn_workspace_bytes(params, is_bwd):
    n = ctypes.c_size_t(0)
    _check(lib.slimpipe_attn_workspace_bytes(ctypes.byref(params), 1 if is_bwd else 0, ctypes.byref(n)), "workspace_bytes")
    return n.value


def _ws(workspace):
    return (workspace.data_ptr(), workspace.numel()) if workspace is not None else (None, 0)


def _outputs(q_slice, out_dtype, out, lse):
    """out and lse of a forward call, allocated where the caller gave none."""
    B, s, Hq, D = q_slice.shape
    if out is None:
        out = torch.empty((B, s, Hq, D), device=q_slice.device, dtype=torch.float32 if out_dtype == F32 else torch.bfloat16)
    if lse is None:
        lse = torch.empty((B, Hq, s), device=q_slice.device, dtype=torch.float32)
    return out, lse


def slimpipe_attn_fwd(q_slice, k_prefix, v_prefix, q_offset, kv_begin, kv_end, causal=True, scale=None,
                      out_dtype=BF16, out=None, lse=None, workspace=None):
    """-> (out, lse).  out [B,s,Hq,D] (bf16 or fp32), lse [B,Hq,s] fp32.  workspace: uint8 tensor the library may
    use to cut a short slice over a long cache into key ranges (slimpipe_attn_workspace_bytes(p, False))."""
    if out is None or lse is None:
        out, lse = _outputs(q_slice, out_dtype, out, lse)
    p = _params(q_slice, k_prefix, out, out, q_offset, kv_begin, kv_end, causal, scale, out_dtype)
    _check(lib.slimpipe_attn_fwd(ctypes.byref(p), q_slice.data_ptr(), k_prefix.data_ptr(), v_prefix.data_ptr(),
                                 out.data_ptr(), lse.data_ptr(), *_ws(workspace), _stream()), "slimpipe_attn_fwd")
    return out, lse


def slimpipe_attn_bwd(q_slice, k_prefix, v_prefix, out, d_out, lse, q_offset, kv_begin, kv_end, dk_acc, dv_acc,
                      causal=True, scale=None, dq=None, dq_dtype=BF16, dq_accumulate=False, dkv_accumulate=True,
                      workspace=None):
    """-> dq.  dk_acc/dv_acc (fp32, shaped like k_prefix) get rows [kv_begin, kv_end) written or incremented."""
    if dq is None:
        dq = torch.empty_like(q_slice, dtype=torch.float32 if dq_dtype == F32 else torch.bfloat16)
    if not (_same_strides(dq, q_slice) and _same_strides(dk_acc, k_prefix) and _same_strides(dv_acc, k_prefix)):
        raise SlimpipeError("dq must have the strides of q; dk_acc/dv_acc those of k")
    p = _params(q_slice, k_prefix, out, d_out, q_offset, kv_begin, kv_end, causal, scale, BF16)
    if workspace is None:
        workspace = torch.empty(slimpipe_attn_workspace_bytes(p, True), device=q_slice.device, dtype=torch.uint8)
    _check(lib.slimpipe_attn_bwd(ctypes.byref(p), q_slice.data_ptr(), k_prefix.data_ptr(), v_prefix.data_ptr(),
                                 out.data_ptr(), d_out.data_ptr(), lse.data_ptr(), dq.data_ptr(), dq_dtype,
                                 1 if dq_accumulate else 0, dk_acc.data_ptr(), dv_acc.data_ptr(),
                                 1 if dkv_accumulate else 0, workspace.data_ptr(), workspace.numel(), _stream()),
           "slimpipe_attn_bwd")
    return dq


def slimpipe_attn_bwd_noalloc(q_slice, k_prefix, v_prefix, out, d_out, lse, q_offset, kv_begin, kv_end, dq, dk_acc, dv_acc,
                              causal=True, scale=None, dq_accumulate=False, dkv_accumulate=True):
    """slimpipe_attn_bwd without a workspace and without any allocation (the binding allocates nothing either: dq is
    the caller's, float32 or bf16 by its dtype).  -> the status code's check; results in dq, dk_acc, dv_acc."""
    if not (_same_strides(dq, q_slice) and _same_strides(dk_acc, k_prefix) and _same_strides(dv_acc, k_prefix)):
        raise SlimpipeError("dq must have the strides of q; dk_acc/dv_acc those of k")
    p = _params(q_slice, k_prefix, out, d_out, q_offset, kv_begin, kv_end, causal, scale, BF16)
    _check(lib.slimpipe_attn_bwd_noalloc(ctypes.byref(p), q_slice.data_ptr(), k_prefix.data_ptr(), v_prefix.data_ptr(),
                                         out.data_ptr(), d_out.data_ptr(), lse.data_ptr(), dq.data_ptr(),
                                         F32 if dq.dtype == torch.float32 else BF16, 1 if dq_accumulate else 0,
                                         dk_acc.data_ptr(), dv_acc.data_ptr(), 1 if dkv_accumulate else 0, _stream()),
           "slimpipe_attn_bwd_noalloc")
    return dq


def _chunk_table(chunks):
    """list of tensors -> ctypes array of device pointers (all chunks share shape and strides)."""
    c0 = chunks[0]
    for c in chunks:
        if c.shape != c0.shape or not _same_strides(c, c0):
            raise SlimpipeError("chunks must share shape and strides")
    return (ctypes.c_void_p * len(chunks))(*[c.data_ptr() for c in chunks])


class _ChunkedKV:
    """What _params needs to know of a chunk list: the shape and strides of the virtual prefix."""
    def __init__(self, chunks):
        c0 = chunks[0]
        self.shape = (c0.shape[0], len(chunks) * c0.shape[1], c0.shape[2], c0.shape[3])
        self._strides = c0.stride()

    def stride(self):
        return self._strides


def slimpipe_attn_fwd_chunked(q_slice, k_chunks, v_chunks, q_offset, kv_begin, kv_end, causal=True, scale=None,
                              out_dtype=BF16, out=None, lse=None, workspace=None):
    """As slimpipe_attn_fwd with K/V given as lists of equally shaped chunks [B, chunk_len, Hkv, D]."""
    if out is None or lse is None:
        out, lse = _outputs(q_slice, out_dtype, out, lse)
    p = _params(q_slice, _ChunkedKV(k_chunks), out, out, q_offset, kv_begin, kv_end, causal, scale, out_dtype)
    _check(lib.slimpipe_attn_fwd_chunked(ctypes.byref(p), q_slice.data_ptr(), _chunk_table(k_chunks), _chunk_table(v_chunks),
                                         len(k_chunks), k_chunks[0].shape[1], out.data_ptr(), lse.data_ptr(), *_ws(workspace),
                                         _stream()),
           "slimpipe_attn_fwd_chunked")
    return out, lse


def slimpipe_attn_fwd_ranges(q_slice, k_chunks, v_chunks, q_offset, ranges, causal=True, scale=None, merged=True,
                             out_dtype=BF16, out=None, lse=None):
    """One launch over several key ranges [(kv_begin, kv_end), ...] of one query slice; k_chunks / v_chunks: a list
    of chunks, or one tensor.  -> (part_out [R,B,s,Hq,D] fp32, part_lse [R,B,Hq,s], out, lse); out and lse are the
    merged result, or None with merged=False."""
    if not isinstance(k_chunks, (list, tuple)):
        k_chunks, v_chunks = [k_chunks], [v_chunks]
    B, s, Hq, D = q_slice.shape
    R = len(ranges)
    part_out = torch.empty((R, B, s, Hq, D), device=q_slice.device, dtype=torch.float32)
    part_lse = torch.empty((R, B, Hq, s), device=q_slice.device, dtype=torch.float32)
    out, lse = _outputs(q_slice, out_dtype, out, lse) if merged else (None, None)
    kv, out_like = _ChunkedKV(k_chunks), out if merged else part_out[0]
    p = _params(q_slice, kv, out_like, out_like, q_offset, 0, kv.shape[1], causal, scale, out_dtype)
    begins = (ctypes.c_int64 * R)(*[int(a) for a, _ in ranges])
    ends = (ctypes.c_int64 * R)(*[int(b) for _, b in ranges])
    _check(lib.slimpipe_attn_fwd_ranges(ctypes.byref(p), q_slice.data_ptr(), _chunk_table(k_chunks), _chunk_table(v_chunks),
                                        len(k_chunks), k_chunks[0].shape[1], R, begins, ends, part_out.data_ptr(), part_lse.data_ptr(),
                                        out.data_ptr() if merged else None, lse.data_ptr() if merged else None, _stream()),
           "slimpipe_attn_fwd_ranges")
    return part_out, part_lse, out, lse


def slimpipe_attn_bwd_chunked(q_slice, k_chunks, v_chunks, out, d_out, lse, q_offset, kv_begin, kv_end, dk_chunks, dv_chunks,
                              causal=True, scale=None, dq=None, dq_dtype=BF16, dq_accumulate=False, dkv_accumulate=True,
                              workspace=None):
    """As slimpipe_attn_bwd with K/V and the fp32 dK/dV accumulators given as lists of chunks."""
    if dq is None:
        dq = torch.empty_like(q_slice, dtype=torch.float32 if dq_dtype == F32 else torch.bfloat16)
    if not _same_strides(dq, q_slice):
        raise SlimpipeError("dq must have the strides of q")
    for c in list(dk_chunks) + list(dv_chunks):
        if not _same_strides(c, k_chunks[0]):
            raise SlimpipeError("dk/dv chunks must have the strides of the k chunks")
    p = _params(q_slice, _ChunkedKV(k_chunks), out, d_out, q_offset, kv_begin, kv_end, causal, scale, BF16)
    if workspace is None:
        workspace = torch.empty(slimpipe_attn_workspace_bytes(p, True), device=q_slice.device, dtype=torch.uint8)
    _check(lib.slimpipe_attn_bwd_chunked(ctypes.byref(p), q_slice.data_ptr(), _chunk_table(k_chunks), _chunk_table(v_chunks),
                                         len(k_chunks), k_chunks[0].shape[1], out.data_ptr(), d_out.data_ptr(), lse.data_ptr(),
                                         dq.data_ptr(), dq_dtype, 1 if dq_accumulate else 0, _chunk_table(dk_chunks),
                                         _chunk_table(dv_chunks), 1 if dkv_accumulate else 0, workspace.data_ptr(),
                                         workspace.numel(), _stream()),
           "slimpipe_attn_bwd_chunked")
    return dq


def slimpipe_attn_merge(outs, lses, out_dtype=BF16, out=None, lse=None):
    """Merge partial (out, lse) pairs over disjoint key sets -> (out, lse)."""
    n = len(outs)
    B, s, Hq, D = outs[0].shape
    part_dtype = F32 if outs[0].dtype == torch.float32 else BF16
    for o in outs:
        if not o.is_contiguous():
            raise SlimpipeError("partial outputs must be contiguous")
    if out is None:
        out = torch.empty((B, s, Hq, D), device=outs[0].device, dtype=torch.float32 if out_dtype == F32 else torch.bfloat16)
    if lse is None:
        lse = torch.empty((B, Hq, s), device=outs[0].device, dtype=torch.float32)
    op = (ctypes.c_void_p * n)(*[o.data_ptr() for o in outs])
    lp = (ctypes.c_void_p * n)(*[l.data_ptr() for l in lses])
    _check(lib.slimpipe_attn_merge(n, op, lp, part_dtype, B, s, Hq, D, out.data_ptr(), out_dtype, lse.data_ptr(), _stream()),
           "slimpipe_attn_merge")
    return out, lse


def slimpipe_attn_finalize_bf16(acc, dst=None):
    if dst is None:
        dst = torch.empty(acc.shape, device=acc.device, dtype=torch.bfloat16)
    _check(lib.slimpipe_attn_finalize_bf16(acc.data_ptr(), dst.data_ptr(), acc.numel(), _stream()), "finalize_bf16")
    return dst


KERNEL_KINDS = ("fwd", "delta", "dq", "dkdv", "merge", "finalize", "dkdv_reduce", "dq_reduce",
                "bwd_both", "both_reduce")


def slimpipe_attn_mfma_rate(random_operands):
    """-> TFLOP/s of a pure bf16 MFMA stream on this GPU (constant or random operands)."""
    sink = torch.zeros(4, device="cuda", dtype=torch.float32)
    tf = ctypes.c_double(0.0)
    _check(lib.slimpipe_attn_mfma_rate(1 if random_operands else 0, sink.data_ptr(), ctypes.byref(tf), _stream()), "mfma_rate")
    return tf.value


def slimpipe_attn_dq_atomic_probe(s_q, heads, key_tiles, rows_per_step, placement, rotate, filler_mfma, with_atomics):
    """-> (ms, every element of dq holds the expected count, workgroups not on XCD w % 8 [placement 1 only])."""
    dq = torch.zeros((s_q, heads, 128), device="cuda", dtype=torch.float32)
    mism = torch.zeros(1, device="cuda", dtype=torch.int32)
    ms = ctypes.c_double(0.0)
    torch.cuda.synchronize()
    rc = lib.slimpipe_attn_dq_atomic_probe(dq.data_ptr(), s_q, heads, key_tiles, rows_per_step, placement, rotate, filler_mfma,
                                           1 if with_atomics else 0, mism.data_ptr(), ctypes.byref(ms), _stream())
    _check(rc, "dq_atomic_probe (step/HIP error %s)" % ms.value)
    want = float(key_tiles * (64 // rows_per_step)) if with_atomics else 0.0
    ok = bool((dq == want).all())
    return ms.value, ok, int(mism.item())


def slimpipe_attn_xcd_rate(iters=20000, rounds=4):
    """-> {xcd: (workgroups, mean workgroup ms, last end ms)} for `rounds` workgroups of equal matrix work per compute unit."""
    n = rounds * torch.cuda.get_device_properties(0).multi_processor_count
    t0 = torch.zeros(n, device="cuda", dtype=torch.int64)
    t1 = torch.zeros(n, device="cuda", dtype=torch.int64)
    xcc = torch.zeros(n, device="cuda", dtype=torch.int32)
    for _ in range(2):          # the second launch is the one reported (clocks settled)
        _check(lib.slimpipe_attn_xcd_rate(iters, n, t0.data_ptr(), t1.data_ptr(), xcc.data_ptr(), _stream()), "xcd_rate")
    t0, t1, xcc = t0.cpu(), t1.cpu(), xcc.cpu()
    base = int(t0.min())
    out = {}
    for x in sorted(set(xcc.tolist())):
        sel = xcc == x
        out[int(x)] = (int(sel.sum()), float((t1[sel] - t0[sel]).double().mean()) / 1e5, float(int(t1[sel].max()) - base) / 1e5)
    return out


def slimpipe_attn_bwd_plan(params, n_chunks, workspace_bytes):
    """How a backward call would be cut into work items with a workspace of that size (host code only)."""
    plan = BwdPlan()
    _check(lib.slimpipe_attn_bwd_plan(ctypes.byref(params), n_chunks, workspace_bytes, ctypes.byref(plan)), "bwd_plan")
    return plan


def slimpipe_attn_call_path(params, is_bwd, n_chunks, workspace_bytes):
    """Which kernels a call with a workspace of that size takes (host code only; forward: 0 bytes = no workspace)."""
    path = CallPath()
    _check(lib.slimpipe_attn_call_path(ctypes.byref(params), 1 if is_bwd else 0, n_chunks, workspace_bytes, ctypes.byref(path)), "call_path")
    return path


def slimpipe_attn_small_bwd_plan(params, n_chunks, workspace_bytes):
    """How the kernel of 32-row and 32-key items would do a backward call that takes it; all zero for others (host code only)."""
    plan = SmallBwdPlan()
    _check(lib.slimpipe_attn_small_bwd_plan(ctypes.byref(params), n_chunks, workspace_bytes, ctypes.byref(plan)), "small_bwd_plan")
    return plan


def slimpipe_attn_profile_enable(enable):
    _check(lib.slimpipe_attn_profile_enable(1 if enable else 0), "profile_enable")


def slimpipe_attn_profile_read():
    """-> {kernel kind: (total ms, launches)} since the last read (waits for the recorded events)."""
    ms = (ctypes.c_double * len(KERNEL_KINDS))()
    n = (ctypes.c_int64 * len(KERNEL_KINDS))()
    _check(lib.slimpipe_attn_profile_read(ms, n), "profile_read")
    return {k: (ms[i], n[i]) for i, k in enumerate(KERNEL_KINDS)}
