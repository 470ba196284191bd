"""ctypes binding of include/moss.h.  Argument marshalling only: every step of the
path runs in the HIP kernels.  torch is used for device memory and streams.

The calls that a training step or a forward pass makes go through _moss_calls first (csrc/moss_calls.cpp), which does in native
code what the functions here do, for plain arguments, and answers None to anything else."""
import ctypes as C
import os
import re

_PKG = os.path.dirname(os.path.abspath(__file__))
# MOSS_HIP_LIBRARY names another build of the same library (the tests load a sanitizer build this way)
_LIB_PATH = os.environ.get("MOSS_HIP_LIBRARY") or os.path.join(_PKG, "libmoss_hip.so")
_HEADER = os.path.join(os.path.dirname(_PKG), "include", "moss.h")
_lib = None

MOSS_DT_BF16, MOSS_DT_F32 = 0, 1
MOSS_Q_ROW, MOSS_Q_COL = 1, 2
MOSS_EXP_NEAREST, MOSS_EXP_CEIL = 0, 4
MOSS_WS_KEPT = 8
MOSS_WSTATE_STEP_MISMATCH = 1


class MossError(RuntimeError):
    pass


class WScaleState(C.Structure):
    _fields_ = [("s_base", C.c_float), ("s_cur", C.c_float), ("cum_lr", C.c_double),
                ("step", C.c_int64), ("last_rebase", C.c_int64),
                ("amax_seen", C.c_float), ("overflow_count", C.c_uint32),
                ("clipped_count", C.c_uint32), ("flags", C.c_uint32)]


class AdamWArgs(C.Structure):
    _fields_ = [("lr", C.c_float), ("beta1", C.c_float), ("beta2", C.c_float),
                ("eps", C.c_float), ("weight_decay", C.c_float),
                ("one_minus_beta1", C.c_float), ("one_minus_beta2", C.c_float),
                ("bias_corr1", C.c_float), ("bias_corr2", C.c_float),
                ("margin", C.c_float), ("interval", C.c_int32), ("step", C.c_int64)]


def lib_path():
    return _LIB_PATH


def exported_symbols():
    """Names of the functions include/moss.h declares."""
    text = open(_HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(moss_[a-z0-9_]+)\s*\(", text)))


def load():
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise MossError(f"{_LIB_PATH} is missing: build it with `python -m paper_2511_05811_amd.build` "
                        "(there is no fallback path)")
    L = C.CDLL(_LIB_PATH)
    vp, i64, u32, sz, ci = C.c_void_p, C.c_int64, C.c_uint, C.c_size_t, C.c_int
    L.moss_status_string.restype = C.c_char_p
    L.moss_status_string.argtypes = [ci]
    L.moss_device_cu_count.restype = ci
    L.moss_quant_workspace_bytes.restype = sz
    L.moss_quant_workspace_bytes.argtypes = [i64, i64, u32]
    L.moss_quant_act_2level.argtypes = [vp, i64, i64, i64, u32, vp, vp, vp, vp, vp, vp, sz, vp]
    L.moss_quant_act_2level_noalloc.argtypes = [vp, i64, i64, i64, u32, vp, vp, vp, vp, vp, vp]
    L.moss_quant_act_2level_given_max.argtypes = [vp, i64, i64, i64, u32, vp, vp, vp, vp, vp, vp, vp]
    L.moss_swiglu_bf16.argtypes = [vp, vp, i64, i64, i64, vp, vp, vp]
    L.moss_swiglu_bf16_backward.argtypes = [vp, vp, vp, i64, i64, i64, vp, vp, vp, vp, vp]
    L.moss_add_rmsnorm_bf16.argtypes = [vp, vp, vp, C.c_float, i64, i64, i64, vp, vp, vp, vp]
    L.moss_rmsnorm_bf16_backward.argtypes = [vp, vp, vp, vp, C.c_float, i64, i64, i64, vp, vp, vp]
    L.moss_quant_set_poll_limit.restype = None
    L.moss_quant_set_poll_limit.argtypes = [u32]
    L.moss_weight_workspace_bytes.restype = sz
    L.moss_weight_workspace_bytes.argtypes = [i64, i64]
    L.moss_weight_autoscale_init.argtypes = [vp, ci, i64, i64, vp, vp, vp, vp, sz, vp]
    L.moss_weight_autoscale_cast.argtypes = [vp, vp, vp, vp, ci, i64, i64, C.POINTER(AdamWArgs), vp, vp, vp, vp, sz, vp]
    L.moss_gemm_workspace_bytes.restype = sz
    L.moss_gemm_workspace_bytes.argtypes = [i64, i64, i64]
    L.moss_gemm_fp8_mx.argtypes = [i64, i64, i64, vp, vp, vp, vp, vp, vp, vp, ci, i64, ci, vp, sz, vp]
    L.moss_gemm_bf16_baseline.argtypes = [i64, i64, i64, vp, vp, vp, i64, vp]
    _lib = L
    return L


def _check(rc, what):
    if rc != 0:
        raise MossError(f"{what}: {load().moss_status_string(rc).decode()} (status {rc})")


_calls = None      # the native calls, bound to the library; False if they have not been built for this torch and this library


def _bind_calls():
    global _calls
    L = load()
    import torch
    names = ("moss_quant_workspace_bytes", "moss_quant_act_2level", "moss_quant_act_2level_given_max", "moss_gemm_fp8_mx",
             "moss_weight_workspace_bytes", "moss_weight_autoscale_cast", "moss_internal_swiglu_bf16", "moss_internal_swiglu_bf16_backward",
             "moss_internal_add_rmsnorm_bf16", "moss_internal_rmsnorm_bf16_backward")     # (these take scratch)
    try:
        from . import _moss_calls as native
        get_device, get_stream = torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream
        addresses = tuple(C.cast(getattr(L, n), C.c_void_p).value for n in names)
        L.moss_internal_interface.restype = C.c_uint32
        built_for_these = native.interface != 0 and (native.torch_version, native.interface) == (torch.__version__, L.moss_internal_interface())
    except (ImportError, AttributeError):
        built_for_these = False
    if not built_for_these:
        _calls = False
        return _calls
    native.bind(addresses, _check, AdamWArgs, get_device, get_stream)
    _calls = native
    return _calls


# What a call costs on the host decides the smallest problems (a GEMM of a few microseconds): pointers go to ctypes as plain
# integers, and the current stream's handle is asked for directly, 0.2 us where a torch.cuda.Stream object takes 2.7 us
# (a GEMM call 8.5 -> 4.6 us, of which 3.5 us are ctypes and the launch).
def _ptr(t):
    return None if t is None else t.data_ptr()


def _stream():
    import torch
    if not torch.cuda.is_initialized():
        torch.cuda.init()
    try:
        return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    except AttributeError:      # a torch without these internal names
        return torch.cuda.current_stream().cuda_stream


def device_cu_count():
    return load().moss_device_cu_count()


def _workspace(nbytes, device):
    import torch
    return torch.empty(max(int(nbytes), 16), dtype=torch.uint8, device=device)


def quant_act_2level(x, flags=MOSS_Q_ROW, out=None, workspace=None):
    """x: torch.bfloat16 [rows, cols] on the GPU (row stride may exceed cols).
    Returns dict(q_row, e_row, q_col, e_col, s) of device tensors (absent outputs are None)."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.quant_act_2level(x, flags, out, workspace)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = x.shape
    assert x.dtype == torch.bfloat16 and x.is_cuda and x.stride(1) == 1
    ld = x.stride(0)
    dev = x.device
    out = out or {}
    u8 = torch.uint8
    want_row, want_col = bool(flags & MOSS_Q_ROW), bool(flags & MOSS_Q_COL)
    q_row = out.get("q_row") if want_row else None
    e_row = out.get("e_row") if want_row else None
    q_col = out.get("q_col") if want_col else None
    e_col = out.get("e_col") if want_col else None
    if want_row and q_row is None:
        q_row = torch.empty((rows, cols), dtype=u8, device=dev)
        e_row = torch.empty((rows, cols // 32), dtype=u8, device=dev)
    if want_col and q_col is None:
        q_col = torch.empty((cols, rows), dtype=u8, device=dev)
        e_col = torch.empty((cols, rows // 32), dtype=u8, device=dev)
    s = out.get("s")
    if s is None:
        s = torch.empty(1, dtype=torch.float32, device=dev)
    if workspace is None:
        workspace = _workspace(L.moss_quant_workspace_bytes(rows, cols, flags), dev)
    rc = L.moss_quant_act_2level(_ptr(x), rows, cols, ld, flags, _ptr(q_row), _ptr(e_row), _ptr(q_col), _ptr(e_col),
                                 _ptr(s), _ptr(workspace), workspace.numel(), _stream())
    _check(rc, "moss_quant_act_2level")
    return dict(q_row=q_row, e_row=e_row, q_col=q_col, e_col=e_col, s=s)


def quant_act_2level_noalloc(x, flags, out):
    """moss_quant_act_2level_noalloc: every output tensor comes from the caller (`out` holds q_row/e_row and/or
    q_col/e_col and s), the scratch is the library's own static array; nothing is allocated."""
    rows, cols = x.shape
    want_row, want_col = bool(flags & MOSS_Q_ROW), bool(flags & MOSS_Q_COL)
    rc = load().moss_quant_act_2level_noalloc(
        _ptr(x), rows, cols, x.stride(0), flags, _ptr(out["q_row"] if want_row else None),
        _ptr(out["e_row"] if want_row else None), _ptr(out["q_col"] if want_col else None),
        _ptr(out["e_col"] if want_col else None), _ptr(out["s"]), _stream())
    _check(rc, "moss_quant_act_2level_noalloc")
    return out


def quant_act_2level_given_max(x, absmax_bits, flags=MOSS_Q_ROW, out=None):
    """quant_act_2level for a tensor whose producer left a bound of max|x| (BF16 magnitude bits) in the
    one-element int32 device tensor `absmax_bits`: one launch, x read once, no workspace."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.quant_act_2level_given_max(x, absmax_bits, flags, out)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = x.shape
    assert x.dtype == torch.bfloat16 and x.is_cuda and x.stride(1) == 1
    assert absmax_bits.dtype == torch.int32 and absmax_bits.is_cuda and absmax_bits.numel() == 1
    dev = x.device
    out = out or {}
    u8 = torch.uint8
    want_row, want_col = bool(flags & MOSS_Q_ROW), bool(flags & MOSS_Q_COL)
    q_row = out.get("q_row") if want_row else None
    e_row = out.get("e_row") if want_row else None
    q_col = out.get("q_col") if want_col else None
    e_col = out.get("e_col") if want_col else None
    if want_row and q_row is None:
        q_row = torch.empty((rows, cols), dtype=u8, device=dev)
        e_row = torch.empty((rows, cols // 32), dtype=u8, device=dev)
    if want_col and q_col is None:
        q_col = torch.empty((cols, rows), dtype=u8, device=dev)
        e_col = torch.empty((cols, rows // 32), dtype=u8, device=dev)
    s = out.get("s")
    if s is None:
        s = torch.empty(1, dtype=torch.float32, device=dev)
    rc = L.moss_quant_act_2level_given_max(_ptr(x), rows, cols, x.stride(0), flags, _ptr(absmax_bits), _ptr(q_row), _ptr(e_row),
                                           _ptr(q_col), _ptr(e_col), _ptr(s), _stream())
    _check(rc, "moss_quant_act_2level_given_max")
    return dict(q_row=q_row, e_row=e_row, q_col=q_col, e_col=e_col, s=s)


def swiglu_bf16(gate, up, h=None, absmax_bits=None):
    """h = silu(gate) * up (BF16) and max|h| as BF16 magnitude bits in a one-element int32 tensor."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.swiglu_bf16(gate, up, h, absmax_bits)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = gate.shape
    for t in (gate, up):
        assert t.dtype == torch.bfloat16 and t.is_cuda and t.stride(1) == 1 and t.shape == gate.shape and t.stride(0) == gate.stride(0)
    if h is None:
        h = torch.empty_strided((rows, cols), (gate.stride(0), 1), dtype=torch.bfloat16, device=gate.device)
    assert h.stride(0) == gate.stride(0) and h.stride(1) == 1
    if absmax_bits is None:
        absmax_bits = torch.empty(1, dtype=torch.int32, device=gate.device)
    rc = L.moss_swiglu_bf16(_ptr(gate), _ptr(up), rows, cols, gate.stride(0), _ptr(h), _ptr(absmax_bits), _stream())
    _check(rc, "moss_swiglu_bf16")
    return h, absmax_bits


def swiglu_bf16_backward(gate, up, dh, d_gate=None, d_up=None, d_gate_absmax_bits=None, d_up_absmax_bits=None):
    """(d_gate, d_up, their maximum words) for the upstream gradient dh of h = silu(gate) * up."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.swiglu_bf16_backward(gate, up, dh, d_gate, d_up, d_gate_absmax_bits, d_up_absmax_bits)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = gate.shape
    ld = gate.stride(0)
    for t in (gate, up, dh):
        assert t.dtype == torch.bfloat16 and t.is_cuda and t.stride(1) == 1 and t.shape == gate.shape and t.stride(0) == ld
    mk = lambda: torch.empty_strided((rows, cols), (ld, 1), dtype=torch.bfloat16, device=gate.device)
    d_gate = mk() if d_gate is None else d_gate
    d_up = mk() if d_up is None else d_up
    assert d_gate.stride(0) == ld and d_up.stride(0) == ld
    if d_gate_absmax_bits is None:
        d_gate_absmax_bits = torch.empty(1, dtype=torch.int32, device=gate.device)
    if d_up_absmax_bits is None:
        d_up_absmax_bits = torch.empty(1, dtype=torch.int32, device=gate.device)
    rc = L.moss_swiglu_bf16_backward(_ptr(gate), _ptr(up), _ptr(dh), rows, cols, ld, _ptr(d_gate), _ptr(d_up),
                                     _ptr(d_gate_absmax_bits), _ptr(d_up_absmax_bits), _stream())
    _check(rc, "moss_swiglu_bf16_backward")
    return d_gate, d_up, d_gate_absmax_bits, d_up_absmax_bits


def add_rmsnorm_bf16(x, gamma, eps, delta=None, h=None, y=None, absmax_bits=None):
    """(h, y, max word): h = x + delta (x itself if delta is None), y = rmsnorm(h) * gamma, max|y| as BF16 bits."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.add_rmsnorm_bf16(x, gamma, eps, delta, h, y, absmax_bits)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = x.shape
    ld = x.stride(0)
    for t in (x, delta):
        assert t is None or (t.dtype == torch.bfloat16 and t.is_cuda and t.stride(1) == 1 and t.shape == x.shape and t.stride(0) == ld)
    assert gamma.dtype == torch.bfloat16 and gamma.is_contiguous() and gamma.shape == (cols,)
    mk = lambda: torch.empty_strided((rows, cols), (ld, 1), dtype=torch.bfloat16, device=x.device)
    if delta is not None and h is None:
        h = mk()
    y = mk() if y is None else y
    if absmax_bits is None:
        absmax_bits = torch.empty(1, dtype=torch.int32, device=x.device)
    rc = L.moss_add_rmsnorm_bf16(_ptr(x), _ptr(delta), _ptr(gamma), float(eps), rows, cols, ld, _ptr(h) if delta is not None else None,
                                 _ptr(y), _ptr(absmax_bits), _stream())
    _check(rc, "moss_add_rmsnorm_bf16")
    return (h if delta is not None else x), y, absmax_bits


def rmsnorm_bf16_backward(h, gamma, dy, eps, d_res=None, d_h=None, absmax_bits=None):
    """(d_h, max word) for the upstream gradient dy of rmsnorm(h) * gamma, plus the residual-path gradient d_res."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.rmsnorm_bf16_backward(h, gamma, dy, eps, d_res, d_h, absmax_bits)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = h.shape
    ld = h.stride(0)
    for t in (h, dy, d_res):
        assert t is None or (t.dtype == torch.bfloat16 and t.is_cuda and t.stride(1) == 1 and t.shape == h.shape and t.stride(0) == ld)
    assert gamma.dtype == torch.bfloat16 and gamma.is_contiguous() and gamma.shape == (cols,)
    if d_h is None:
        d_h = torch.empty_strided((rows, cols), (ld, 1), dtype=torch.bfloat16, device=h.device)
    if absmax_bits is None:
        absmax_bits = torch.empty(1, dtype=torch.int32, device=h.device)
    rc = L.moss_rmsnorm_bf16_backward(_ptr(h), _ptr(gamma), _ptr(dy), _ptr(d_res), float(eps), rows, cols, ld, _ptr(d_h),
                                      _ptr(absmax_bits), _stream())
    _check(rc, "moss_rmsnorm_bf16_backward")
    return d_h, absmax_bits


def quant_set_poll_limit(polls):
    """Bound of the one-launch quantizer's wait for the grid-wide maximum (0: slow path)."""
    load().moss_quant_set_poll_limit(int(polls))


def new_wscale_state(device):
    import torch
    return torch.zeros(C.sizeof(WScaleState), dtype=torch.uint8, device=device)


def read_wscale_state(state):
    """Copy the device-resident state struct to the host (synchronizes)."""
    return WScaleState.from_buffer_copy(bytes(state.cpu().numpy().tobytes()))


def _dt(t):
    import torch
    if t.dtype == torch.float32:
        return MOSS_DT_F32
    if t.dtype == torch.bfloat16:
        return MOSS_DT_BF16
    raise MossError(f"unsupported dtype {t.dtype}")


def weight_autoscale_init(w, state, wq=None, wq_t=None, want_transpose=False, workspace=None):
    import torch
    L = load()
    rows, cols = w.shape
    assert w.is_cuda and w.is_contiguous()
    if wq is None:
        wq = torch.empty((rows, cols), dtype=torch.uint8, device=w.device)
    if want_transpose and wq_t is None:
        wq_t = torch.empty((cols, rows), dtype=torch.uint8, device=w.device)
    if workspace is None:
        workspace = _workspace(L.moss_weight_workspace_bytes(rows, cols), w.device)
    rc = L.moss_weight_autoscale_init(_ptr(w), _dt(w), rows, cols, _ptr(state), _ptr(wq), _ptr(wq_t),
                                      _ptr(workspace), workspace.numel(), _stream())
    _check(rc, "moss_weight_autoscale_init")
    return wq, wq_t


def weight_autoscale_cast(w, m, v, g, args, state, wq=None, wq_t=None, want_transpose=False, workspace=None):
    """One fused AdamW + scale prediction + FP8 cast step; w, m, v float32 in place."""
    native = _bind_calls() if _calls is None else _calls
    if native:
        done = native.weight_autoscale_cast(w, m, v, g, args, state, wq, wq_t, want_transpose, workspace)
        if done is not None:
            return done
    import torch
    L = load()
    rows, cols = w.shape
    for t in (w, m, v):
        assert t.is_cuda and t.is_contiguous() and t.dtype == torch.float32
    assert g.is_cuda and g.is_contiguous()
    if wq is None:
        wq = torch.empty((rows, cols), dtype=torch.uint8, device=w.device)
    if want_transpose and wq_t is None:
        wq_t = torch.empty((cols, rows), dtype=torch.uint8, device=w.device)
    if workspace is None:
        workspace = _workspace(L.moss_weight_workspace_bytes(rows, cols), w.device)
    rc = L.moss_weight_autoscale_cast(_ptr(w), _ptr(m), _ptr(v), _ptr(g), _dt(g), rows, cols, C.byref(args),
                                      _ptr(state), _ptr(wq), _ptr(wq_t), _ptr(workspace), workspace.numel(), _stream())
    _check(rc, "moss_weight_autoscale_cast")
    return wq, wq_t


def gemm_fp8_mx(a_q, a_e, a_s, b_q, b_e, b_s, out=None, out_dtype=None, accumulate=False):
    """out[m,n] (+)= a_s*b_s*sum_k a[m,k] 2^(ae-127) b[n,k] 2^(be-127); a_q [M,K], b_q [N,K] uint8 device tensors,
    a_e/b_e uint8 [.,K/32] or None, a_s/b_s float32 device scalars."""
    native = _bind_calls() if _calls is None else _calls
    if native and (out_dtype is None or out is not None):
        done = native.gemm_fp8_mx(a_q, a_e, a_s, b_q, b_e, b_s, out, accumulate)
        if done is not None:
            return done
    import torch
    L = load()
    M, K = a_q.shape
    N = b_q.shape[0]
    assert b_q.shape[1] == K and a_q.is_contiguous() and b_q.is_contiguous()
    if out is None:
        out = torch.empty((M, N), dtype=out_dtype or torch.bfloat16, device=a_q.device)
    rc = L.moss_gemm_fp8_mx(M, N, K, _ptr(a_q), _ptr(a_e), _ptr(a_s), _ptr(b_q), _ptr(b_e), _ptr(b_s),
                            _ptr(out), _dt(out), out.stride(0), int(bool(accumulate)), None, 0, _stream())
    _check(rc, "moss_gemm_fp8_mx")
    return out


def gemm_bf16_baseline(a, b, out=None):
    import torch
    L = load()
    M, K = a.shape
    N = b.shape[0]
    assert a.dtype == torch.bfloat16 and b.dtype == torch.bfloat16 and a.is_contiguous() and b.is_contiguous()
    if out is None:
        out = torch.empty((M, N), dtype=torch.bfloat16, device=a.device)
    rc = L.moss_gemm_bf16_baseline(M, N, K, _ptr(a), _ptr(b), _ptr(out), out.stride(0), _stream())
    _check(rc, "moss_gemm_bf16_baseline")
    return out
