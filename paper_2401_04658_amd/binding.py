"""Thin binding of libla2.so: argument marshalling only.  The calls of the path go through the native module _la2_native
(csrc/la2_python.cpp: checks, output tensors, descriptors), queries and tuning knobs through ctypes.

Every step of the path runs in the library's HIP kernels; there is no CPU or
PyTorch fallback.  torch is used for device memory and streams.  If the shared
library is missing the first call raises (build it with
`python -m paper_2401_04658_amd.build` or `__graft_entry__.build()`).
"""
import ctypes
import importlib.machinery
import importlib.util
import os
import sys

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libla2.so")
_NATIVE_PATH = os.path.join(_HERE, "_la2_native.so")
_lib = None
_native = None

LA2_F32, LA2_BF16, LA2_F16 = 0, 1, 2
LA2_OP_FWD, LA2_OP_BWD, LA2_OP_FWD_STATE, LA2_OP_BWD_STATE = 0, 1, 2, 3


class LA2Error(RuntimeError):
    def __init__(self, code, message):
        super().__init__("la2 status %d: %s" % (code, message))
        self.code = code


class la2_desc(ctypes.Structure):
    _fields_ = [
        ("batch", ctypes.c_int32), ("heads", ctypes.c_int32), ("seqlen", ctypes.c_int32),
        ("head_dim", ctypes.c_int32), ("dtype", ctypes.c_int32), ("reserved", ctypes.c_int32),
        ("stride_b", ctypes.c_int64), ("stride_h", ctypes.c_int64), ("stride_n", ctypes.c_int64),
    ]


def lib_path():
    return _LIB_PATH


def load():
    """Loads libla2.so (no fallback: raises if it has not been built).  The argument types are those of the whole C ABI, for programs
    and tests that call it through ctypes; the functions below go through the native module but for queries and knobs."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise FileNotFoundError(
            "%s not found: the HIP library has not been built (python -m paper_2401_04658_amd.build)" % _LIB_PATH)
    lib = ctypes.CDLL(_LIB_PATH)
    vp, sz, i32 = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int32
    dp = ctypes.POINTER(la2_desc)
    lib.la2_desc_dense.argtypes = [dp, i32, i32, i32, i32, i32]
    lib.la2_desc_dense.restype = None
    lib.la2_workspace_bytes.argtypes = [dp, i32]
    lib.la2_workspace_bytes.restype = sz
    lib.la2_chunk_plan.argtypes = [dp, ctypes.POINTER(i32), ctypes.POINTER(i32)]
    lib.la2_chunk_plan.restype = ctypes.c_int
    lib.la2_block_size.argtypes = [dp]
    lib.la2_block_size.restype = i32
    lib.la2_set_chunk_tokens.argtypes = [i32]
    lib.la2_set_chunk_tokens.restype = None
    lib.la2_set_scan_variant.argtypes = [i32]
    lib.la2_set_scan_variant.restype = None
    lib.la2_fwd_state_norm.argtypes = [dp, vp, vp, vp, vp, vp, ctypes.c_float, vp, vp, vp, vp, sz, vp]
    lib.la2_fwd_state_norm.restype = ctypes.c_int
    lib.la2_bwd_state_norm.argtypes = [dp] + [vp] * 15 + [sz, vp]
    lib.la2_bwd_state_norm.restype = ctypes.c_int
    lib.la2_decode_step_norm.argtypes = [i32, i32, i32, i32, vp, vp, vp, vp, vp, ctypes.c_float, vp, vp]
    lib.la2_decode_step_norm.restype = ctypes.c_int
    lib.la2_fwd.argtypes = [dp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_fwd.restype = ctypes.c_int
    lib.la2_fwd_noalloc.argtypes = [dp, vp, vp, vp, vp, vp, vp]
    lib.la2_fwd_noalloc.restype = ctypes.c_int
    lib.la2_bwd.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_bwd.restype = ctypes.c_int
    lib.la2_fwd_state.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_fwd_state.restype = ctypes.c_int
    lib.la2_bwd_state.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_bwd_state.restype = ctypes.c_int
    lib.la2_bwd_saved.argtypes = [dp] + [vp] * 12 + [sz, i32, vp, sz, vp]
    lib.la2_bwd_saved.restype = ctypes.c_int
    lib.la2_fwd_norm.argtypes = [dp, vp, vp, vp, vp, ctypes.c_float, vp, vp, vp, sz, vp]
    lib.la2_fwd_norm.restype = ctypes.c_int
    lib.la2_bwd_norm.argtypes = [dp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_bwd_norm.restype = ctypes.c_int
    lib.la2_varlen_workspace_bytes.argtypes = [dp, ctypes.c_int64, i32]
    lib.la2_varlen_workspace_bytes.restype = sz
    lib.la2_fwd_varlen.argtypes = [dp, vp, ctypes.c_int64, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_fwd_varlen.restype = ctypes.c_int
    lib.la2_bwd_varlen.argtypes = [dp, vp, ctypes.c_int64, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_bwd_varlen.restype = ctypes.c_int
    lib.la2_fwd_varlen_state.argtypes = [dp, vp, ctypes.c_int64, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.la2_fwd_varlen_state.restype = ctypes.c_int
    lib.la2_bwd_varlen_state.argtypes = [dp, vp, ctypes.c_int64] + [vp] * 11 + [vp, sz, vp]
    lib.la2_bwd_varlen_state.restype = ctypes.c_int
    lib.la2_fwd_varlen_norm.argtypes = [dp, vp, ctypes.c_int64, vp, vp, vp, vp, ctypes.c_float, vp, vp, vp, sz, vp]
    lib.la2_fwd_varlen_norm.restype = ctypes.c_int
    lib.la2_bwd_varlen_norm.argtypes = [dp, vp, ctypes.c_int64] + [vp] * 11 + [vp, sz, vp]
    lib.la2_bwd_varlen_norm.restype = ctypes.c_int
    lib.la2_decode_multi_norm.argtypes = [i32, i32, i32, i32, i32, vp, vp, vp, vp, vp, ctypes.c_float, vp, vp, vp]
    lib.la2_decode_multi_norm.restype = ctypes.c_int
    lib.la2_left_product_fwd.argtypes = [dp, vp, vp, vp, vp, vp, vp]
    lib.la2_left_product_fwd.restype = ctypes.c_int
    lib.la2_left_product_bwd.argtypes = [dp] + [vp] * 9
    lib.la2_left_product_bwd.restype = ctypes.c_int
    lib.la2_decode_multi.argtypes = [i32, i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, vp]
    lib.la2_decode_multi.restype = ctypes.c_int
    lib.la2_decode_step.argtypes = [i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, vp]
    lib.la2_decode_step.restype = ctypes.c_int
    lib.la2_status_string.argtypes = [ctypes.c_int]
    lib.la2_status_string.restype = ctypes.c_char_p
    _lib = lib
    return lib


def _module():
    """The native module (no fallback: raises if it has not been built)."""
    global _native
    if _native is None:
        if not os.path.exists(_NATIVE_PATH):
            raise FileNotFoundError(
                "%s not found: the native module has not been built (python -m paper_2401_04658_amd.build)" % _NATIVE_PATH)
        here = sys.version_info[:2] + (str(torch.__version__),)
        try:
            loader = importlib.machinery.ExtensionFileLoader("_la2_native", _NATIVE_PATH)
            spec = importlib.util.spec_from_file_location("_la2_native", _NATIVE_PATH, loader=loader)
            module = importlib.util.module_from_spec(spec)
            loader.exec_module(module)
        except ImportError as e:   # (a torch without a function that it calls, among others)
            raise ImportError("%s does not load with Python %d.%d and torch %s; build it with them (python -m paper_2401_04658_amd.build): %s"
                              % ((_NATIVE_PATH,) + here + (e,))) from e
        built = getattr(module, "built_for", None)
        if built != here:
            raise ImportError("%s was built for %s, not for Python %d.%d and torch %s; build it again (python -m paper_2401_04658_amd.build)"
                              % ((_NATIVE_PATH, "Python %d.%d and torch %s" % built if built else "another torch") + here))
        _native = module
    return _native


def _check(code):
    if code != 0:
        raise LA2Error(code, load().la2_status_string(code).decode())


def _dtype_code(t):
    if t.dtype == torch.bfloat16:
        return LA2_BF16
    if t.dtype == torch.float16:
        return LA2_F16
    if t.dtype == torch.float32:
        return LA2_F32
    raise TypeError("la2: dtype must be torch.bfloat16, torch.float16 or torch.float32, got %s" % t.dtype)


def make_desc(t):
    """Descriptor of a [batch, heads, seqlen, head_dim] tensor (feature stride must be 1)."""
    if t.dim() != 4:
        raise ValueError("la2: expected a [batch, heads, seqlen, head_dim] tensor")
    if t.shape[3] > 1 and t.stride(3) != 1:
        raise ValueError("la2: the feature dimension must be contiguous")
    b, h, n, d = t.shape
    return la2_desc(b, h, n, d, _dtype_code(t), 0, t.stride(0), t.stride(1), t.stride(2))


# The stream handle and the device number are taken from where torch.cuda.current_stream and torch.cuda.device take them (a
# torch without these two: from the wrappers), and the device is switched only if it has to be (decode, batch 1: 11.0 us a call
# with the wrappers, 7.5 without).
_current_device = getattr(torch._C, "_cuda_getDevice", None) or torch.cuda.current_device
_current_stream = (getattr(torch._C, "_cuda_getCurrentRawStream", None)
                   or (lambda device: torch.cuda.current_stream(device).cuda_stream))


def _run(entry, t, *args):
    """entry(*args, stream) on the current stream of t's device, which is made the current device."""
    device = t.get_device()
    if device == _current_device():
        code = entry(*args, _current_stream(device))
    else:
        with torch.cuda.device(device):
            code = entry(*args, _current_stream(device))
    if code:
        _check(code)


def _on_gpu(t, name):
    if not t.is_cuda:
        raise ValueError("%s: tensors must live on the GPU" % name)


def _outputs(lib, q, out):
    """dq, dk, dv: the caller's or new ones."""
    if out is None:
        return lib.like(q), lib.like(q), lib.like(q)
    dq, dk, dv = out
    lib.same_layout(q, dq, dk, dv)
    return dq, dk, dv


def la2_workspace_bytes(t, op=LA2_OP_FWD):
    desc = make_desc(t)
    return int(load().la2_workspace_bytes(ctypes.byref(desc), op))


def la2_chunk_plan(t):
    """(nchunks, chunk_tokens) of the sequence chunks la2_fwd / la2_bwd run in parallel for this tensor."""
    desc = make_desc(t)
    n, c = ctypes.c_int32(0), ctypes.c_int32(0)
    _check(load().la2_chunk_plan(ctypes.byref(desc), ctypes.byref(n), ctypes.byref(c)))
    return int(n.value), int(c.value)


def la2_block_size(t):
    desc = make_desc(t)
    return int(load().la2_block_size(ctypes.byref(desc)))


def la2_set_chunk_tokens(tokens):
    load().la2_set_chunk_tokens(int(tokens))


def la2_set_scan_variant(variant):
    load().la2_set_scan_variant(int(variant))


def la2_fwd(q, k, v, lam, out=None, workspace=None):
    """o = LA2(q, k, v; lam) on the GPU.  q, k, v: [b, H, n, d] bf16/fp32; lam: fp32 [H] (device)."""
    lib = _module()
    _on_gpu(q, "la2_fwd")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    ws = lib.workspace(q, LA2_OP_FWD) if workspace is None else workspace
    _run(lib.la2_fwd, q, q, q, k, v, lam, out, ws, ws)
    return out


def la2_fwd_noalloc(q, k, v, lam, out):
    """la2_fwd into `out` with the library's built-in scratch instead of a workspace; the call itself allocates
    nothing (so `out` is required)."""
    lib = _module()
    _on_gpu(q, "la2_fwd_noalloc")
    lib.given(lam)
    lib.same_layout(q, k, v, out)
    _run(lib.la2_fwd_noalloc, q, q, q, k, v, lam, out)
    return out


def la2_bwd(q, k, v, d_o, lam, out=None, workspace=None):
    """(dq, dk, dv) of sum(o * d_o) on the GPU."""
    lib = _module()
    _on_gpu(q, "la2_bwd")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    ws = lib.workspace(q, LA2_OP_BWD) if workspace is None else workspace
    _run(lib.la2_bwd, q, q, q, k, v, d_o, lam, dq, dk, dv, ws, ws)
    return dq, dk, dv


def _rstd(lib, rstd, q, shape, name, what):
    """The caller's row scales, checked, or new ones."""
    if rstd is None:
        return lib.f32(q, *shape)
    if rstd.dtype != torch.float32 or tuple(rstd.shape) != shape or not rstd.is_contiguous():
        raise ValueError("%s: rstd must be a contiguous fp32 %s tensor" % (name, what))
    return rstd


def la2_fwd_norm(q, k, v, lam, eps=1e-6, out=None, rstd=None, workspace=None):
    """(o, rstd) = Norm(LA2(q, k, v; lam)): every output row scaled by rstd = 1 / sqrt(mean(row^2) + eps)."""
    lib = _module()
    _on_gpu(q, "la2_fwd_norm")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    rstd = _rstd(lib, rstd, q, tuple(q.shape[:3]), "la2_fwd_norm", "[batch, heads, seqlen]")
    ws = lib.workspace(q, LA2_OP_FWD) if workspace is None else workspace
    _run(lib.la2_fwd_norm, q, q, q, k, v, lam, eps, out, rstd, ws, ws)
    return out, rstd


def _given_rstd(lib, rstd, q, shape, name, what):
    if rstd is None:
        raise ValueError("%s: rstd is the forward call's" % name)
    return _rstd(lib, rstd, q, shape, name, what)


def la2_bwd_norm(q, k, v, o, rstd, d_o, lam, out=None, d_u=None, workspace=None):
    """(dq, dk, dv) of sum(la2_fwd_norm(q, k, v)[0] * d_o); o, rstd are la2_fwd_norm's results.  d_u (same
    layout as d_o) receives the gradient with respect to the un-normalised output."""
    lib = _module()
    _on_gpu(q, "la2_bwd_norm")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v, o, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    if d_u is None:
        d_u = lib.like(q)
    else:
        lib.same_layout(q, d_u)
    _given_rstd(lib, rstd, q, tuple(q.shape[:3]), "la2_bwd_norm", "[batch, heads, seqlen]")
    ws = lib.workspace(q, LA2_OP_BWD) if workspace is None else workspace
    _run(lib.la2_bwd_norm, q, q, q, k, v, o, rstd, d_o, lam, d_u, dq, dk, dv, ws, ws)
    return dq, dk, dv


def _varlen_desc(q, cu_seqlens, max_seqlen):
    """Descriptor of packed sequences: q is [total_positions, heads, head_dim], cu_seqlens int32 [batch + 1]."""
    if q.dim() != 3 or q.stride(2) != 1:
        raise ValueError("la2: packed tensors are [total_positions, heads, head_dim] with unit feature stride")
    if cu_seqlens.dtype != torch.int32 or cu_seqlens.dim() != 1 or not cu_seqlens.is_contiguous() or not cu_seqlens.is_cuda:
        raise ValueError("la2: cu_seqlens must be a contiguous int32 vector on the GPU")
    return la2_desc(cu_seqlens.numel() - 1, q.shape[1], int(max_seqlen), q.shape[2], _dtype_code(q), 0,
                    0, q.stride(1), q.stride(0))


def _varlen_workspace(q, desc, op, workspace):
    need = int(load().la2_varlen_workspace_bytes(ctypes.byref(desc), q.shape[0], op))
    if need == 0:
        return None
    if workspace is None:
        return torch.empty(need, dtype=torch.uint8, device=q.device)
    if workspace.numel() * workspace.element_size() < need:
        raise ValueError("la2: workspace too small (%d < %d bytes)" % (workspace.numel() * workspace.element_size(), need))
    return workspace


def la2_fwd_varlen(q, k, v, lam, cu_seqlens, max_seqlen, out=None, workspace=None):
    """o for packed sequences of different lengths: q, k, v [total_positions, heads, head_dim]; sequence b is
    positions cu_seqlens[b] .. cu_seqlens[b + 1] - 1; max_seqlen bounds the lengths."""
    lib = _module()
    _on_gpu(q, "la2_fwd_varlen")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    desc = _varlen_desc(q, cu_seqlens, max_seqlen)
    ws = _varlen_workspace(q, desc, LA2_OP_FWD, workspace)
    _run(lib.la2_fwd_varlen, q, desc, cu_seqlens, q.shape[0], q, k, v, lam, out, ws, ws)
    return out


def la2_bwd_varlen(q, k, v, d_o, lam, cu_seqlens, max_seqlen, out=None, workspace=None):
    """(dq, dk, dv) for packed sequences of different lengths (see la2_fwd_varlen)."""
    lib = _module()
    _on_gpu(q, "la2_bwd_varlen")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    desc = _varlen_desc(q, cu_seqlens, max_seqlen)
    ws = _varlen_workspace(q, desc, LA2_OP_BWD, workspace)
    _run(lib.la2_bwd_varlen, q, desc, cu_seqlens, q.shape[0], q, k, v, d_o, lam, dq, dk, dv, ws, ws)
    return dq, dk, dv


def la2_fwd_varlen_state(q, k, v, lam, cu_seqlens, max_seqlen, kv_init=None, want_final=True, out=None, kv_final=None,
                         workspace=None):
    """Packed sequences as segments: o and every sequence's state after its last position, each started from its
    kv_init (fp32 [sequences, H, d, d], None = zero).  Returns (o, kv_final or None)."""
    lib = _module()
    _on_gpu(q, "la2_fwd_varlen_state")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    desc = _varlen_desc(q, cu_seqlens, max_seqlen)
    nseq = desc.batch
    if not want_final:
        kv_final = None
    elif kv_final is None:
        kv_final = lib.f32(q, nseq, q.shape[1], q.shape[2], q.shape[2])
    ws = _varlen_workspace(q, desc, LA2_OP_FWD, workspace)
    _run(lib.la2_fwd_varlen_state, q, desc, cu_seqlens, q.shape[0], q, k, v, lam, lib.state(kv_init, q, "kv_init", nseq), out,
         lib.state(kv_final, q, "kv_final", nseq), ws, ws)
    return out, kv_final


def la2_bwd_varlen_state(q, k, v, d_o, lam, cu_seqlens, max_seqlen, kv_init=None, d_kv_final=None, want_d_kv_init=True,
                         out=None, d_kv_init=None, workspace=None):
    """Backward of la2_fwd_varlen_state.  Returns (dq, dk, dv, d_kv_init or None)."""
    lib = _module()
    _on_gpu(q, "la2_bwd_varlen_state")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    desc = _varlen_desc(q, cu_seqlens, max_seqlen)
    nseq = desc.batch
    if not want_d_kv_init:
        d_kv_init = None
    elif d_kv_init is None:
        d_kv_init = lib.f32(q, nseq, q.shape[1], q.shape[2], q.shape[2])
    ws = _varlen_workspace(q, desc, LA2_OP_BWD, workspace)
    _run(lib.la2_bwd_varlen_state, q, desc, cu_seqlens, q.shape[0], q, k, v, d_o, lam, lib.state(kv_init, q, "kv_init", nseq),
         lib.state(d_kv_final, q, "d_kv_final", nseq), dq, dk, dv, lib.state(d_kv_init, q, "d_kv_init", nseq), ws, ws)
    return dq, dk, dv, d_kv_init


def la2_fwd_varlen_norm(q, k, v, lam, cu_seqlens, max_seqlen, eps=1e-6, out=None, rstd=None, workspace=None):
    """(o, rstd) of the normalised operator over packed sequences; rstd is fp32 [heads, total_positions]."""
    lib = _module()
    _on_gpu(q, "la2_fwd_varlen_norm")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    rstd = _rstd(lib, rstd, q, (q.shape[1], q.shape[0]), "la2_fwd_varlen_norm", "[heads, total_positions]")
    desc = _varlen_desc(q, cu_seqlens, max_seqlen)
    ws = _varlen_workspace(q, desc, LA2_OP_FWD, workspace)
    _run(lib.la2_fwd_varlen_norm, q, desc, cu_seqlens, q.shape[0], q, k, v, lam, eps, out, rstd, ws, ws)
    return out, rstd


def la2_bwd_varlen_norm(q, k, v, o, rstd, d_o, lam, cu_seqlens, max_seqlen, out=None, d_u=None, workspace=None):
    """(dq, dk, dv) of the normalised operator over packed sequences (o, rstd from la2_fwd_varlen_norm)."""
    lib = _module()
    _on_gpu(q, "la2_bwd_varlen_norm")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v, o, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    if d_u is None:
        d_u = lib.like(q)
    else:
        lib.same_layout(q, d_u)
    _given_rstd(lib, rstd, q, (q.shape[1], q.shape[0]), "la2_bwd_varlen_norm", "[heads, total_positions]")
    desc = _varlen_desc(q, cu_seqlens, max_seqlen)
    ws = _varlen_workspace(q, desc, LA2_OP_BWD, workspace)
    _run(lib.la2_bwd_varlen_norm, q, desc, cu_seqlens, q.shape[0], q, k, v, o, rstd, d_o, lam, d_u, dq, dk, dv, ws, ws)
    return dq, dk, dv


def la2_fwd_state(q, k, v, lam, kv_init=None, want_final=True, out=None, kv_final=None, workspace=None):
    """One segment of a sequence: o and the state after its last position, started from kv_init
    (fp32 [b, H, d, d], None = zero).  Returns (o, kv_final or None)."""
    lib = _module()
    _on_gpu(q, "la2_fwd_state")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    b, h, _, d = q.shape
    if not want_final:
        kv_final = None
    elif kv_final is None:
        kv_final = lib.f32(q, b, h, d, d)
    ws = lib.workspace(q, LA2_OP_FWD_STATE) if workspace is None else workspace
    _run(lib.la2_fwd_state, q, q, q, k, v, lam, lib.state(kv_init, q, "kv_init"), out, lib.state(kv_final, q, "kv_final"), ws, ws)
    return out, kv_final


def la2_bwd_state(q, k, v, d_o, lam, kv_init=None, d_kv_final=None, want_d_kv_init=True, out=None,
                  d_kv_init=None, workspace=None, fwd_workspace=None, fwd_wrote_kv_final=False):
    """Backward of one segment.  Returns (dq, dk, dv, d_kv_init or None).  fwd_workspace: the workspace
    tensor the forward call used (contents untouched since), to reuse its chunk states; fwd_wrote_kv_final:
    whether that call handed out kv_final."""
    lib = _module()
    _on_gpu(q, "la2_bwd_state")
    lib.given(lam, workspace, fwd_workspace)
    lib.same_layout(q, k, v, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    b, h, _, d = q.shape
    if not want_d_kv_init:
        d_kv_init = None
    elif d_kv_init is None:
        d_kv_init = lib.f32(q, b, h, d, d)
    ws = lib.workspace(q, LA2_OP_BWD_STATE) if workspace is None else workspace
    _run(lib.la2_bwd_saved, q, q, q, k, v, d_o, lam, lib.state(kv_init, q, "kv_init"), lib.state(d_kv_final, q, "d_kv_final"),
         dq, dk, dv, lib.state(d_kv_init, q, "d_kv_init"), fwd_workspace, fwd_workspace, 1 if fwd_wrote_kv_final else 0, ws, ws)
    return dq, dk, dv, d_kv_init


def la2_fwd_state_norm(q, k, v, lam, eps=1e-6, kv_init=None, want_final=True, out=None, rstd=None, kv_final=None,
                       workspace=None):
    """la2_fwd_norm on one segment of a sequence, started from kv_init.  Returns (o, rstd, kv_final or None)."""
    lib = _module()
    _on_gpu(q, "la2_fwd_state_norm")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    b, h, n, d = q.shape
    rstd = _rstd(lib, rstd, q, (b, h, n), "la2_fwd_state_norm", "[batch, heads, seqlen]")
    if not want_final:
        kv_final = None
    elif kv_final is None:
        kv_final = lib.f32(q, b, h, d, d)
    ws = lib.workspace(q, LA2_OP_FWD_STATE) if workspace is None else workspace
    _run(lib.la2_fwd_state_norm, q, q, q, k, v, lam, lib.state(kv_init, q, "kv_init"), eps, out, rstd,
         lib.state(kv_final, q, "kv_final"), ws, ws)
    return out, rstd, kv_final


def la2_bwd_state_norm(q, k, v, o, rstd, d_o, lam, kv_init=None, d_kv_final=None, want_d_kv_init=True, out=None,
                       d_u=None, d_kv_init=None, workspace=None):
    """Backward of la2_fwd_state_norm.  Returns (dq, dk, dv, d_kv_init or None)."""
    lib = _module()
    _on_gpu(q, "la2_bwd_state_norm")
    lib.given(lam, workspace)
    lib.same_layout(q, k, v, o, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    if d_u is None:
        d_u = lib.like(q)
    else:
        lib.same_layout(q, d_u)
    b, h, n, d = q.shape
    _given_rstd(lib, rstd, q, (b, h, n), "la2_bwd_state_norm", "[batch, heads, seqlen]")
    if not want_d_kv_init:
        d_kv_init = None
    elif d_kv_init is None:
        d_kv_init = lib.f32(q, b, h, d, d)
    ws = lib.workspace(q, LA2_OP_BWD_STATE) if workspace is None else workspace
    _run(lib.la2_bwd_state_norm, q, q, q, k, v, o, rstd, d_o, lam, lib.state(kv_init, q, "kv_init"),
         lib.state(d_kv_final, q, "d_kv_final"), d_u, dq, dk, dv, lib.state(d_kv_init, q, "d_kv_init"), ws, ws)
    return dq, dk, dv, d_kv_init


def la2_decode_step(q, k, v, lam, kv_state, out=None):
    """One recurrent step; kv_state (fp32 [b, H, d, d]) is updated in place, returns o [b, H, d]."""
    lib = _module()
    _on_gpu(q, "la2_decode_step")
    b, h, d, dtype = lib.decode_shape("la2_decode_step", 3, q, k, v, kv_state, lam, out)
    if out is None:
        out = lib.like(q)
    _run(lib.la2_decode_step, q, b, h, d, dtype, q, k, v, lam, kv_state, out)
    return out


def la2_decode_multi(q, k, v, lam, kv_state, out=None):
    """ntokens consecutive recurrent steps in one launch.  q, k, v: dense [b, H, T, d]; kv_state (fp32
    [b, H, d, d]) is updated in place; returns o [b, H, T, d]."""
    lib = _module()
    _on_gpu(q, "la2_decode_multi")
    b, h, t, d, dtype = lib.decode_shape("la2_decode_multi", 4, q, k, v, kv_state, lam, out)
    if out is None:
        out = lib.like(q)
    _run(lib.la2_decode_multi, q, b, h, d, t, dtype, q, k, v, lam, kv_state, out)
    return out


def la2_decode_step_norm(q, k, v, lam, kv_state, eps=1e-6, out=None):
    """One recurrent step of the normalised operator; kv_state (fp32 [b, H, d, d]) is updated in place, returns
    the normalised o [b, H, d]."""
    lib = _module()
    _on_gpu(q, "la2_decode_step_norm")
    b, h, d, dtype = lib.decode_shape("la2_decode_step_norm", 3, q, k, v, kv_state, lam, out)
    if out is None:
        out = lib.like(q)
    _run(lib.la2_decode_step_norm, q, b, h, d, dtype, q, k, v, lam, kv_state, eps, out)
    return out


def la2_decode_multi_norm(q, k, v, lam, kv_state, eps=1e-6, out=None, rstd=None):
    """ntokens consecutive steps of the normalised operator in one launch; returns (o, rstd [b, H, T])."""
    lib = _module()
    _on_gpu(q, "la2_decode_multi_norm")
    b, h, t, d, dtype = lib.decode_shape("la2_decode_multi_norm", 4, q, k, v, kv_state, lam, out, rstd)
    if out is None:
        out = lib.like(q)
    if rstd is None:
        rstd = lib.f32(q, b, h, t)
    _run(lib.la2_decode_multi_norm, q, b, h, d, t, dtype, q, k, v, lam, kv_state, eps, out, rstd)
    return out, rstd


def la2_left_product_fwd(q, k, v, lam, out=None):
    """The forward pass as the O(n^2 d) masked left product (comparison kernel, bf16)."""
    lib = _module()
    _on_gpu(q, "la2_left_product_fwd")
    lib.given(lam)
    lib.same_layout(q, k, v)
    if out is None:
        out = lib.like(q)
    else:
        lib.same_layout(q, out)
    _run(lib.la2_left_product_fwd, q, q, q, k, v, lam, out)
    return out


def la2_left_product_bwd(q, k, v, d_o, lam, out=None):
    """(dq, dk, dv) as O(n^2 d) masked products (comparison kernel, bf16)."""
    lib = _module()
    _on_gpu(q, "la2_left_product_bwd")
    lib.given(lam)
    lib.same_layout(q, k, v, d_o)
    dq, dk, dv = _outputs(lib, q, out)
    _run(lib.la2_left_product_bwd, q, q, q, k, v, d_o, lam, dq, dk, dv)
    return dq, dk, dv
