"""Thin ctypes binding of libselkv.so (C ABI in include/selkv.h).

Argument marshalling only: every step runs in the HIP kernels of the
library.  Tensors are torch device tensors (PyTorch provides device memory
and the current stream); the functions check dtype, shape, device and
contiguity, then pass raw pointers.  Importing this module raises if the
built library is missing -- there is no fallback path.
"""
from __future__ import annotations

import ctypes
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libselkv.so")

F32, BF16 = 0, 1
GATE_COSINE, GATE_DROP, GATE_MERGE_ALL = 0, 1, 2
ROUTE_BUCKET, ROUTE_FULL_COSINE, ROUTE_BUCKET_NEAREST, ROUTE_COATTN = 0, 1, 2, 3
SELECT_PER_HEAD, SELECT_UNION = 0, 1
ABI_VERSION = 6
CALL_SCORE, CALL_SELECT, CALL_MERGE, CALL_BIAS, CALL_DECODE, CALL_ROUTE, CALL_MERGE_BIAS = range(7)
STATUS = {0: "SELKV_OK", 1: "SELKV_EINVAL", 2: "SELKV_EDTYPE", 3: "SELKV_EUNSUPPORTED", 4: "SELKV_EALIGN",
          5: "SELKV_EWORKSPACE", 6: "SELKV_EHIP"}
GATE_MODES = {"cosine": GATE_COSINE, "drop": GATE_DROP, "merge_all": GATE_MERGE_ALL}
ROUTE_MODES = {"bucket": ROUTE_BUCKET, "full_cosine": ROUTE_FULL_COSINE, "bucket_nearest": ROUTE_BUCKET_NEAREST,
               "coattn": ROUTE_COATTN}
SELECT_MODES = {"per_head": SELECT_PER_HEAD, "union": SELECT_UNION}


class SelkvError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {STATUS.get(status, status)}")


class Params(ctypes.Structure):
    _fields_ = [
        ("struct_size", ctypes.c_uint32),
        ("batch", ctypes.c_int32),
        ("n_heads_kv", ctypes.c_int32),
        ("group", ctypes.c_int32),
        ("head_dim", ctypes.c_int32),
        ("seq_len", ctypes.c_int32),
        ("window", ctypes.c_int32),
        ("pool_kernel", ctypes.c_int32),
        ("recent", ctypes.c_int32),
        ("bucket", ctypes.c_int32),
        ("kv_dtype", ctypes.c_int32),
        ("gate_mode", ctypes.c_int32),
        ("route_mode", ctypes.c_int32),
        ("scale", ctypes.c_float),
        ("alpha", ctypes.c_float),
        ("gate_threshold", ctypes.c_float),
        ("gate_temperature", ctypes.c_float),
        ("budget_ratio", ctypes.c_double),
        ("select_mode", ctypes.c_int32),
        ("merge_keys", ctypes.c_int32),
    ]


def _load():
    if not os.path.exists(LIB_PATH):
        raise ImportError(f"{LIB_PATH} is not built; run paper_2607_16213_amd.build.build() first")
    lib = ctypes.CDLL(LIB_PATH)
    vp, sz, i32, fp, ip = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p
    P = ctypes.POINTER(Params)
    sigs = {
        "selkv_params_init": (None, [P]),
        "selkv_budget": (ctypes.c_int, [P, ctypes.POINTER(i32), ctypes.POINTER(i32), ctypes.POINTER(i32)]),
        "selkv_workspace_size": (ctypes.c_int, [P, i32, i32, ctypes.POINTER(sz)]),
        "selkv_score": (ctypes.c_int, [P, vp, vp, vp, fp, fp, fp, vp, sz, vp]),
        "selkv_select": (ctypes.c_int, [P, fp, ip, ip, vp, sz, vp]),
        "selkv_route_coattn": (ctypes.c_int, [P, vp, vp, ip, ip, ip, vp, sz, vp]),
        "selkv_merge": (ctypes.c_int, [P, vp, vp, fp, fp, ip, ip, vp, vp, ip, fp, vp, sz, vp]),
        "selkv_bias": (ctypes.c_int, [P, fp, ip, ip, ip, fp, fp, vp, sz, vp]),
        "selkv_merge_bias": (ctypes.c_int, [P, vp, vp, fp, fp, ip, ip, vp, vp, ip, fp, fp, vp, sz, vp]),
        "selkv_decode_attn": (ctypes.c_int, [P, vp, vp, vp, fp, i32, fp, vp, sz, vp]),
        "selkv_decode_attn_noalloc": (ctypes.c_int, [P, vp, vp, vp, fp, i32, fp, vp]),
        "selkv_rope_reposition": (ctypes.c_int, [P, ip, vp, ctypes.c_double, vp]),
        "selkv_decode_append": (ctypes.c_int, [P, vp, vp, vp, vp, vp, fp, i32, i32, fp, vp, sz, vp]),
        "selkv_status_string": (ctypes.c_char_p, [ctypes.c_int]),
        "selkv_abi_version": (ctypes.c_int32, []),
    }
    for name, (res, args) in sigs.items():
        f = getattr(lib, name)
        f.restype = res
        f.argtypes = args
    return lib


lib = _load()
if lib.selkv_abi_version() != ABI_VERSION:
    raise ImportError(f"{LIB_PATH} has ABI version {lib.selkv_abi_version()}, this binding expects {ABI_VERSION}")


def params(**kw) -> Params:
    """selkv_params with the paper's defaults, overridden by keyword."""
    p = Params()
    lib.selkv_params_init(ctypes.byref(p))
    for k, v in kw.items():
        if k == "gate_mode" and isinstance(v, str):
            v = GATE_MODES[v]
        if k == "route_mode" and isinstance(v, str):
            v = ROUTE_MODES[v]
        if k == "select_mode" and isinstance(v, str):
            v = SELECT_MODES[v]
        if k == "kv_dtype" and isinstance(v, (str, torch.dtype)):
            v = BF16 if v in ("bf16", torch.bfloat16) else F32
        if not hasattr(p, k):
            raise AttributeError(k)
        setattr(p, k, v)
    return p


def _check(status: int, where: str):
    if status != 0:
        raise SelkvError(status, where)


def budget(p: Params):
    m, mr, ms = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
    _check(lib.selkv_budget(ctypes.byref(p), ctypes.byref(m), ctypes.byref(mr), ctypes.byref(ms)), "selkv_budget")
    return m.value, mr.value, ms.value


def workspace_bytes(p: Params, call: int, cache_len: int = 0) -> int:
    b = ctypes.c_size_t()
    _check(lib.selkv_workspace_size(ctypes.byref(p), call, cache_len, ctypes.byref(b)), "selkv_workspace_size")
    return b.value


def workspace(p: Params, call: int, device, cache_len: int = 0) -> torch.Tensor:
    """Scratch for `call` (zero-filled for tidiness; no call needs it initialised)."""
    nbytes = workspace_bytes(p, call, cache_len)
    return torch.zeros(max(nbytes, 1), dtype=torch.uint8, device=device)


def _ptr(t):
    return None if t is None else t.data_ptr()


# Handle of the current device's current stream (0 is the null stream), without
# building a torch Stream object per call.  A torch without GPU support has no
# such entry, and no call here gets as far as asking for a stream.
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream(stream):
    return _raw_stream(torch.cuda.current_device()) if stream is None else stream.cuda_stream


def _dev(t: torch.Tensor, shape, dtype, name):
    if not t.is_cuda:
        raise ValueError(f"{name} must be a device tensor")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if dtype is not None and t.dtype != dtype:
        raise ValueError(f"{name} has dtype {t.dtype}, expected {dtype}")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
    return t


def _ok(t, shape, dtype):
    """Whether t passes _dev; the calls test this first and say what is wrong only when something is."""
    return t.is_cuda and t.dtype == dtype and t.shape == shape and t.is_contiguous()


def _sizes(p):
    """(m, m_r') of a valid problem, as selkv_budget gives them: m = floor(rho n) in IEEE double.  The library
    validates p itself, so a call on an invalid p fails there (or on a shape) and _refuse says why."""
    try:
        m = int(p.budget_ratio * p.seq_len)
    except (ValueError, OverflowError):   # rho is not a number
        budget(p)
        raise
    return m, min(p.recent, m)


def _refuse(p, status, where):
    budget(p)                             # an invalid problem is reported as such
    raise SelkvError(status, where)


def _nbytes(ws):
    """Size in bytes of a workspace tensor (any dtype), 0 for none."""
    if ws is None:
        return 0
    if not ws.is_cuda or not ws.is_contiguous():
        raise ValueError("workspace must be a contiguous device tensor")
    return ws.numel() * ws.element_size()


def _kvdt(p: Params):
    return torch.bfloat16 if p.kv_dtype == BF16 else torch.float32


_F32, _I32 = torch.float32, torch.int32


def score(p, K, V, Qwin, score_out, attn, vnorm, ws, stream=None):
    B, H, n, d = p.batch, p.n_heads_kv, p.seq_len, p.head_dim
    m, mr = _sizes(p)
    dt = _kvdt(p)
    kv, q, sc, per_key = (B, H, n, d), (B, H * p.group, p.window, d), (B, H, n - mr), (B, H, n)
    if not (_ok(K, kv, dt) and _ok(V, kv, dt) and _ok(Qwin, q, dt) and _ok(score_out, sc, _F32)
            and _ok(attn, per_key, _F32) and _ok(vnorm, per_key, _F32)):
        budget(p)
        _dev(K, kv, dt, "K"); _dev(V, kv, dt, "V"); _dev(Qwin, q, dt, "Qwin"); _dev(score_out, sc, _F32, "score")
        _dev(attn, per_key, _F32, "attn"); _dev(vnorm, per_key, _F32, "vnorm")
    st = lib.selkv_score(p, K.data_ptr(), V.data_ptr(), Qwin.data_ptr(), score_out.data_ptr(), attn.data_ptr(),
                         vnorm.data_ptr(), _ptr(ws), _nbytes(ws), _stream(stream))
    if st:
        _refuse(p, st, "selkv_score")


def select(p, score_in, kept, evicted, ws=None, stream=None):
    B, H, n = p.batch, p.n_heads_kv, p.seq_len
    m, mr = _sizes(p)
    sc, k, e = (B, H, n - mr), (B, H, m), (B, H, n - m)
    if not (_ok(score_in, sc, _F32) and _ok(kept, k, _I32) and _ok(evicted, e, _I32)):
        budget(p)
        _dev(score_in, sc, _F32, "score"); _dev(kept, k, _I32, "kept_idx"); _dev(evicted, e, _I32, "evicted_idx")
    st = lib.selkv_select(p, score_in.data_ptr(), kept.data_ptr(), evicted.data_ptr(), _ptr(ws), _nbytes(ws),
                          _stream(stream))
    if st:
        _refuse(p, st, "selkv_select")


def route_coattn(p, K, Qwin, kept, evicted, target, ws, stream=None):
    """Co-attention routing (route_mode COATTN): target slots for selkv_merge / selkv_bias."""
    B, H, n, d = p.batch, p.n_heads_kv, p.seq_len, p.head_dim
    m, mr = _sizes(p)
    dt = _kvdt(p)
    kv, q, k, e = (B, H, n, d), (B, H * p.group, p.window, d), (B, H, m), (B, H, n - m)
    if not (_ok(K, kv, dt) and _ok(Qwin, q, dt) and _ok(kept, k, _I32) and _ok(evicted, e, _I32)
            and _ok(target, e, _I32)):
        budget(p)
        _dev(K, kv, dt, "K"); _dev(Qwin, q, dt, "Qwin"); _dev(kept, k, _I32, "kept_idx")
        _dev(evicted, e, _I32, "evicted_idx"); _dev(target, e, _I32, "target")
    st = lib.selkv_route_coattn(p, K.data_ptr(), Qwin.data_ptr(), kept.data_ptr(), evicted.data_ptr(),
                                target.data_ptr(), _ptr(ws), _nbytes(ws), _stream(stream))
    if st:
        _refuse(p, st, "selkv_route_coattn")


def _check_merge(p, K, V, attn, vnorm, kept, evicted, K_out, V_out, target, gate, bias_out=None):
    B, H, n, d = p.batch, p.n_heads_kv, p.seq_len, p.head_dim
    m, mr = _sizes(p)
    dt = _kvdt(p)
    kv, per_key, k, e, out = (B, H, n, d), (B, H, n), (B, H, m), (B, H, n - m), (B, H, m, d)
    if not (_ok(K, kv, dt) and _ok(V, kv, dt) and _ok(attn, per_key, _F32) and _ok(vnorm, per_key, _F32)
            and _ok(kept, k, _I32) and _ok(evicted, e, _I32) and _ok(K_out, out, dt) and _ok(V_out, out, dt)
            and _ok(target, e, _I32) and _ok(gate, e, _F32) and (bias_out is None or _ok(bias_out, k, _F32))):
        budget(p)
        _dev(K, kv, dt, "K"); _dev(V, kv, dt, "V")
        _dev(attn, per_key, _F32, "attn"); _dev(vnorm, per_key, _F32, "vnorm")
        _dev(kept, k, _I32, "kept_idx"); _dev(evicted, e, _I32, "evicted_idx")
        _dev(K_out, out, dt, "K_out"); _dev(V_out, out, dt, "V_out")
        _dev(target, e, _I32, "target"); _dev(gate, e, _F32, "gate")
        if bias_out is not None:
            _dev(bias_out, k, _F32, "bias")


def merge(p, K, V, attn, vnorm, kept, evicted, K_out, V_out, target, gate, ws, stream=None):
    _check_merge(p, K, V, attn, vnorm, kept, evicted, K_out, V_out, target, gate)
    st = lib.selkv_merge(p, K.data_ptr(), V.data_ptr(), attn.data_ptr(), vnorm.data_ptr(), kept.data_ptr(),
                         evicted.data_ptr(), K_out.data_ptr(), V_out.data_ptr(), target.data_ptr(), gate.data_ptr(),
                         _ptr(ws), _nbytes(ws), _stream(stream))
    if st:
        _refuse(p, st, "selkv_merge")


def merge_bias(p, K, V, attn, vnorm, kept, evicted, K_out, V_out, target, gate, bias_out, ws, stream=None):
    """selkv_merge and selkv_bias in one pass (the bias from the merge's own sums)."""
    if bias_out is None:
        raise AttributeError("bias_out must be a device tensor")
    _check_merge(p, K, V, attn, vnorm, kept, evicted, K_out, V_out, target, gate, bias_out)
    st = lib.selkv_merge_bias(p, K.data_ptr(), V.data_ptr(), attn.data_ptr(), vnorm.data_ptr(), kept.data_ptr(),
                              evicted.data_ptr(), K_out.data_ptr(), V_out.data_ptr(), target.data_ptr(),
                              gate.data_ptr(), bias_out.data_ptr(), _ptr(ws), _nbytes(ws), _stream(stream))
    if st:
        _refuse(p, st, "selkv_merge_bias")


def bias(p, attn, kept, evicted, target, gate, bias_out, ws, stream=None):
    B, H, n = p.batch, p.n_heads_kv, p.seq_len
    m, mr = _sizes(p)
    per_key, k, e = (B, H, n), (B, H, m), (B, H, n - m)
    if not (_ok(attn, per_key, _F32) and _ok(kept, k, _I32) and _ok(evicted, e, _I32) and _ok(target, e, _I32)
            and _ok(gate, e, _F32) and _ok(bias_out, k, _F32)):
        budget(p)
        _dev(attn, per_key, _F32, "attn")
        _dev(kept, k, _I32, "kept_idx"); _dev(evicted, e, _I32, "evicted_idx")
        _dev(target, e, _I32, "target"); _dev(gate, e, _F32, "gate")
        _dev(bias_out, k, _F32, "bias")
    st = lib.selkv_bias(p, attn.data_ptr(), kept.data_ptr(), evicted.data_ptr(), target.data_ptr(), gate.data_ptr(),
                        bias_out.data_ptr(), _ptr(ws), _nbytes(ws), _stream(stream))
    if st:
        _refuse(p, st, "selkv_bias")


def rope_reposition(p, kept, K_out, rope_theta, stream=None):
    B, H, d = p.batch, p.n_heads_kv, p.head_dim
    m, mr, ms = budget(p)
    _dev(kept, (B, H, m), _I32, "kept_idx")
    _dev(K_out, (B, H, m, d), _kvdt(p), "K_out")
    _check(lib.selkv_rope_reposition(p, _ptr(kept), _ptr(K_out), float(rope_theta), _stream(stream)),
           "selkv_rope_reposition")


def _check_decode(p, q, K, V, bias_in, out):
    B, H, d = p.batch, p.n_heads_kv, p.head_dim
    L = K.shape[2]
    dt = _kvdt(p)
    qs, kv = (B, H * p.group, d), (B, H, L, d)
    if not (_ok(q, qs, dt) and _ok(K, kv, dt) and _ok(V, kv, dt) and _ok(out, qs, _F32)
            and (bias_in is None or _ok(bias_in, (B, H, L), _F32))):
        _dev(q, qs, dt, "q")
        _dev(K, kv, dt, "K"); _dev(V, kv, dt, "V")
        if bias_in is not None:
            _dev(bias_in, (B, H, L), _F32, "bias")
        _dev(out, qs, _F32, "out")
    return L


def decode_attn(p, q, K, V, bias_in, out, ws, stream=None):
    L = _check_decode(p, q, K, V, bias_in, out)
    st = lib.selkv_decode_attn(p, q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(bias_in), L, out.data_ptr(),
                               _ptr(ws), _nbytes(ws), _stream(stream))
    if st:
        raise SelkvError(st, "selkv_decode_attn")


def decode_attn_noalloc(p, q, K, V, bias_in, out, stream=None):
    """selkv_decode_attn with the library's fixed per-GPU scratch instead of a
    workspace (nothing is allocated; calls overlapping on one GPU race)."""
    L = _check_decode(p, q, K, V, bias_in, out)
    st = lib.selkv_decode_attn_noalloc(p, q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(bias_in), L, out.data_ptr(),
                                       _stream(stream))
    if st:
        raise SelkvError(st, "selkv_decode_attn_noalloc")


def decode_append(p, q, k_new, v_new, K, V, bias_io, cache_len, out, ws, stream=None):
    """Append (k_new, v_new) at entry cache_len (bias 0 there) and attend over
    cache_len + 1 entries; K, V [B, H, capacity, d] and bias [B, H, capacity]."""
    B, H, d = p.batch, p.n_heads_kv, p.head_dim
    cap = K.shape[2]
    dt = _kvdt(p)
    qs, new, kv = (B, H * p.group, d), (B, H, d), (B, H, cap, d)
    if not (_ok(q, qs, dt) and _ok(k_new, new, dt) and _ok(v_new, new, dt) and _ok(K, kv, dt) and _ok(V, kv, dt)
            and _ok(out, qs, _F32) and (bias_io is None or _ok(bias_io, (B, H, cap), _F32))):
        _dev(q, qs, dt, "q")
        _dev(k_new, new, dt, "k_new"); _dev(v_new, new, dt, "v_new")
        _dev(K, kv, dt, "K"); _dev(V, kv, dt, "V")
        if bias_io is not None:
            _dev(bias_io, (B, H, cap), _F32, "bias")
        _dev(out, qs, _F32, "out")
    st = lib.selkv_decode_append(p, q.data_ptr(), k_new.data_ptr(), v_new.data_ptr(), K.data_ptr(), V.data_ptr(),
                                 _ptr(bias_io), int(cache_len), cap, out.data_ptr(), _ptr(ws), _nbytes(ws),
                                 _stream(stream))
    if st:
        raise SelkvError(st, "selkv_decode_append")


class Compressor:
    """Owns the output and scratch tensors of one problem size and runs the
    compression calls (score, select, [route_coattn,] merge_bias, or merge then
    bias with fused=False) on the current stream.  Allocation happens once, in
    the constructor."""

    def __init__(self, p: Params, device):
        self.p = p
        B, H, n, d = p.batch, p.n_heads_kv, p.seq_len, p.head_dim
        self.m, self.mr, self.ms = budget(p)
        m, mr = self.m, self.mr
        dt = _kvdt(p)
        f32, i32 = torch.float32, torch.int32
        self.score = torch.empty((B, H, n - mr), dtype=f32, device=device)
        self.attn = torch.empty((B, H, n), dtype=f32, device=device)
        self.vnorm = torch.empty((B, H, n), dtype=f32, device=device)
        self.kept = torch.empty((B, H, m), dtype=i32, device=device)
        self.evicted = torch.empty((B, H, n - m), dtype=i32, device=device)
        self.K_out = torch.empty((B, H, m, d), dtype=dt, device=device)
        self.V_out = torch.empty((B, H, m, d), dtype=dt, device=device)
        self.target = torch.empty((B, H, n - m), dtype=i32, device=device)
        self.gate = torch.empty((B, H, n - m), dtype=f32, device=device)
        self.bias = torch.empty((B, H, m), dtype=f32, device=device)
        self.ws_score = workspace(p, CALL_SCORE, device)
        self.ws_select = workspace(p, CALL_SELECT, device)
        self.ws_merge = workspace(p, CALL_MERGE_BIAS, device)   # covers merge and bias alone too
        self.ws_route = workspace(p, CALL_ROUTE, device) if p.route_mode == ROUTE_COATTN else None

    def run(self, K, V, Qwin, stream=None, fused=True):
        p = self.p
        score(p, K, V, Qwin, self.score, self.attn, self.vnorm, self.ws_score, stream)
        select(p, self.score, self.kept, self.evicted, self.ws_select, stream)
        if p.route_mode == ROUTE_COATTN:
            route_coattn(p, K, Qwin, self.kept, self.evicted, self.target, self.ws_route, stream)
        if fused:
            merge_bias(p, K, V, self.attn, self.vnorm, self.kept, self.evicted, self.K_out, self.V_out, self.target,
                       self.gate, self.bias, self.ws_merge, stream)
        else:
            merge(p, K, V, self.attn, self.vnorm, self.kept, self.evicted, self.K_out, self.V_out, self.target,
                  self.gate, self.ws_merge, stream)
            bias(p, self.attn, self.kept, self.evicted, self.target, self.gate, self.bias, self.ws_merge, stream)
        return self

    def outputs(self):
        return dict(score=self.score, attn=self.attn, vnorm=self.vnorm, kept=self.kept, evicted=self.evicted,
                    K_out=self.K_out, V_out=self.V_out, target=self.target, gate=self.gate, bias=self.bias)


class Decoder:
    """Owns the split-K workspace for decode over caches of `cache_len` entries."""

    def __init__(self, p: Params, cache_len: int, device):
        self.p = p
        self.cache_len = cache_len
        self.ws = workspace(p, CALL_DECODE, device, cache_len)
        self.out = torch.empty((p.batch, p.n_heads_kv * p.group, p.head_dim), dtype=torch.float32, device=device)

    def run(self, q, K, V, bias_in=None, out=None, stream=None):
        o = self.out if out is None else out
        decode_attn(self.p, q, K, V, bias_in, o, self.ws, stream)
        return o
