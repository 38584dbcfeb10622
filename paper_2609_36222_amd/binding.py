"""ctypes binding of libbase.so (the C ABI in include/base.h).

Argument marshalling only: torch tensors in, raw device pointers and sizes
out, the caller's current HIP stream, and a Python exception for a negative
status.  Every step of the computation runs in the library's HIP kernels.
The library must be built (``paper_2609_36222_amd.build``); loading fails
loudly otherwise -- there is no fallback.
"""
from __future__ import annotations

import ctypes
import os

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "_lib", "libbase.so")

BASE_F32, BASE_BF16 = 0, 1
W_ROWMAJOR, W_PACKED = 0, 1
GATE_PAPER, GATE_RENORM = 0, 1
FILL_BACKFILL, FILL_DROP = 0, 2
SCORE_BASE, SCORE_TOP1, SCORE_WEIGHT, SCORE_WEIGHT_SQ, SCORE_STATIC = 0, 1, 2, 3, 4

EXPORTS = ("base_workspace_bytes", "base_route", "base_predict_cost",
           "base_select", "base_moe_forward", "base_decode_layer",
           "base_decode_layer_noalloc",
           "base_pack_experts", "base_set_stage_events", "base_layer_stages",
           "base_status_string",
           "base_calib_stats_bytes", "base_calib_ws_bytes", "base_calib_reset",
           "base_calib_accumulate")
CALIB_LIB_PATH = os.path.join(HERE, "_lib", "libbase_calib.so")
N_STAGES = 9     # one kernel each; base_set_stage_events takes 2 events per stage
STAGES = ("scores", "tail", "select", "backfill", "compact", "gather",
          "ffn_gateup", "ffn_down", "combine")

_vp = ctypes.c_void_p
_i32 = ctypes.c_int32


class base_layer(ctypes.Structure):
    _fields_ = [("d", _i32), ("E", _i32), ("K", _i32), ("I", _i32),
                ("dtype", _i32), ("norm_topk", _i32), ("w_layout", _i32),
                ("score_rule", _i32), ("w_router", _vp), ("b_router", _vp), ("pred_a", _vp),
                ("pred_b", _vp), ("w13", _vp), ("w2", _vp),
                ("n_shared", _i32), ("w13_shared", _vp), ("w2_shared", _vp),
                ("shared_gate", _vp)]


_PLAN_FIELDS = ["logits", "topk_ids", "topk_w", "cost", "scores", "counts",
                "sel_ids", "n_sel", "slot_of_expert", "exec_ids", "exec_gates",
                "offsets", "pair_tok", "pair_gate", "pair_of"]


class base_plan(ctypes.Structure):
    _fields_ = [(f, _vp) for f in _PLAN_FIELDS]


class BaseError(RuntimeError):
    def __init__(self, status, msg):
        super().__init__(f"{msg} (status {status})")
        self.status = status


_lib = None


def load(path: str = LIB_PATH):
    """Load libbase.so; raises if it has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    # torch first: libbase.so then binds to the HIP runtime torch loaded
    # (same SONAME), so streams and events are shared with torch
    import torch  # noqa: F401
    if not os.path.exists(path):
        raise ImportError(
            f"{path} is missing: build it with "
            "`python -m paper_2609_36222_amd.build` (no CPU fallback exists)")
    L = ctypes.CDLL(path)
    L.base_workspace_bytes.restype = ctypes.c_size_t
    L.base_workspace_bytes.argtypes = [ctypes.POINTER(base_layer), _i32, _i32]
    L.base_route.restype = _i32
    L.base_route.argtypes = [ctypes.POINTER(base_layer), _vp, _i32, _vp, _vp,
                             _vp, _vp]
    L.base_predict_cost.restype = _i32
    L.base_predict_cost.argtypes = [ctypes.POINTER(base_layer), _vp, _i32,
                                    _vp, _vp, _vp, _vp]
    L.base_select.restype = _i32
    L.base_select.argtypes = [ctypes.POINTER(base_layer), _i32, _vp, _vp,
                              _i32, _vp, _vp, _vp, _vp, _vp, _vp]
    L.base_moe_forward.restype = _i32
    L.base_moe_forward.argtypes = [ctypes.POINTER(base_layer), _vp, _i32, _vp,
                                   _vp, _vp, _vp, _vp, _i32, _i32, _vp, _vp,
                                   ctypes.POINTER(base_plan), _vp,
                                   ctypes.c_size_t, _vp]
    L.base_decode_layer.restype = _i32
    L.base_decode_layer.argtypes = [ctypes.POINTER(base_layer), _vp, _i32,
                                    _i32, _i32, _vp, _vp,
                                    ctypes.POINTER(base_plan), _vp,
                                    ctypes.c_size_t, _vp]
    L.base_decode_layer_noalloc.restype = _i32
    L.base_decode_layer_noalloc.argtypes = [ctypes.POINTER(base_layer), _vp, _i32,
                                            _i32, _i32, _vp, _vp,
                                            ctypes.POINTER(base_plan), _vp]
    L.base_pack_experts.restype = _i32
    L.base_pack_experts.argtypes = [ctypes.POINTER(base_layer), _vp, _vp, _vp]
    L.base_set_stage_events.restype = _i32
    L.base_set_stage_events.argtypes = [ctypes.POINTER(ctypes.c_void_p), _i32]
    L.base_layer_stages.restype = _i32
    L.base_layer_stages.argtypes = [ctypes.POINTER(base_layer), _i32, _i32,
                                    ctypes.POINTER(_i32)]
    L.base_status_string.restype = ctypes.c_char_p
    L.base_status_string.argtypes = [_i32]
    L.base_calib_stats_bytes.restype = ctypes.c_size_t
    L.base_calib_stats_bytes.argtypes = [ctypes.POINTER(base_layer)]
    L.base_calib_ws_bytes.restype = ctypes.c_size_t
    L.base_calib_ws_bytes.argtypes = [ctypes.POINTER(base_layer), _i32]
    L.base_calib_reset.restype = _i32
    L.base_calib_reset.argtypes = [ctypes.POINTER(base_layer), _vp, _vp]
    L.base_calib_accumulate.restype = _i32
    L.base_calib_accumulate.argtypes = [ctypes.POINTER(base_layer), _vp, _i32, _vp, _vp,
                                        ctypes.c_size_t, _vp]
    _lib = L
    return L


_calib = None


def load_calib(path: str = CALIB_LIB_PATH):
    """Load libbase_calib.so (the predictor fit, base_calib.h)."""
    global _calib
    if _calib is not None:
        return _calib
    load()
    if not os.path.exists(path):
        raise ImportError(f"{path} is missing: build it with "
                          "`python -m paper_2609_36222_amd.build`")
    L = ctypes.CDLL(path)
    L.base_calib_fit.restype = _i32
    L.base_calib_fit.argtypes = [ctypes.POINTER(base_layer), _vp, _i32,
                                 ctypes.POINTER(ctypes.c_double), _vp, _vp, _vp, _vp]
    _calib = L
    return L


def status_string(status: int) -> str:
    return load().base_status_string(int(status)).decode()


def _check(status):
    if status != 0:
        raise BaseError(status, status_string(status))


def _ptr(t):
    """Device pointer of a tensor (None -> NULL)."""
    if t is None:
        return None
    return t.data_ptr()


def _stream(stream):
    import torch
    if stream is None:
        stream = torch.cuda.current_stream()
    return ctypes.c_void_p(stream.cuda_stream)


class Layer:
    """One MoE layer: torch tensors plus the C descriptor pointing at them.

    w_router, b_router, pred_a, pred_b: fp32; w13 [E,2I,d], w2 [E,d,I]:
    fp32 or bf16 (the layer dtype, also the dtype of x and y).  shared:
    None or (w13_shared [S,2I,d], w2_shared [S,d,I], gate [d] fp32 or
    None), the always-active shared experts."""

    def __init__(self, w_router, b_router, pred_a, pred_b, w13, w2,
                 norm_topk: int = 1, w_layout: int = 0, score_rule: int = 0,
                 shared=None):
        import torch
        E, d = w_router.shape
        I = w2.shape[2]
        K = None
        self.tensors = (w_router, b_router, pred_a, pred_b, w13, w2)
        self.dtype = BASE_BF16 if w13.dtype == torch.bfloat16 else BASE_F32
        self.torch_dtype = w13.dtype
        self.d, self.E, self.I, self.K = d, E, I, K
        self.norm_topk = norm_topk
        self.w_layout = w_layout
        self.score_rule = score_rule
        self.shared = shared
        self._desc = None

    def desc(self, K: int) -> base_layer:
        w_router, b_router, pred_a, pred_b, w13, w2 = self.tensors
        return base_layer(self.d, self.E, K, self.I, self.dtype,
                          self.norm_topk, self.w_layout, self.score_rule,
                          _ptr(w_router), _ptr(b_router),
                          _ptr(pred_a), _ptr(pred_b), _ptr(w13), _ptr(w2),
                          *self._shared_fields())

    def _shared_fields(self):
        if self.shared is None:
            return (0, None, None, None)
        w13s, w2s, gate = self.shared
        return (int(w13s.shape[0]), _ptr(w13s), _ptr(w2s), _ptr(gate))


def base_workspace_bytes(desc: base_layer, B: int, budget: int) -> int:
    return int(load().base_workspace_bytes(ctypes.byref(desc), B, budget))


def base_route(desc, x, B, logits, topk_ids, topk_w, stream=None):
    _check(load().base_route(ctypes.byref(desc), _ptr(x), B, _ptr(logits),
                             _ptr(topk_ids), _ptr(topk_w), _stream(stream)))


def base_predict_cost(desc, x, B, topk_ids, topk_w, cost, stream=None):
    _check(load().base_predict_cost(ctypes.byref(desc), _ptr(x), B,
                                    _ptr(topk_ids), _ptr(topk_w), _ptr(cost),
                                    _stream(stream)))


def base_select(desc, B, topk_ids, cost, budget, scores, counts, sel_ids,
                n_sel, slot_of_expert, stream=None):
    _check(load().base_select(ctypes.byref(desc), B, _ptr(topk_ids),
                              _ptr(cost), budget, _ptr(scores), _ptr(counts),
                              _ptr(sel_ids), _ptr(n_sel),
                              _ptr(slot_of_expert), _stream(stream)))


def base_moe_forward(desc, x, B, logits, topk_ids, sel_ids, n_sel,
                     slot_of_expert, budget, flags, residual, y, ws,
                     plan=None, stream=None):
    """Returns the filled base_plan (device pointers into ws)."""
    plan = base_plan() if plan is None else plan
    _check(load().base_moe_forward(
        ctypes.byref(desc), _ptr(x), B, _ptr(logits), _ptr(topk_ids),
        _ptr(sel_ids), _ptr(n_sel), _ptr(slot_of_expert), budget, flags,
        _ptr(residual), _ptr(y), ctypes.byref(plan), _ptr(ws),
        ws.numel() * ws.element_size(), _stream(stream)))
    return plan


def base_decode_layer(desc, x, B, budget, flags, residual, y, ws, plan=None,
                      stream=None):
    """Returns the filled base_plan (device pointers into ws)."""
    plan = base_plan() if plan is None else plan
    _check(load().base_decode_layer(
        ctypes.byref(desc), _ptr(x), B, budget, flags, _ptr(residual), _ptr(y),
        ctypes.byref(plan), _ptr(ws), ws.numel() * ws.element_size(),
        _stream(stream)))
    return plan


def base_decode_layer_noalloc(desc, x, B, budget, flags, residual, y, plan=None,
                              stream=None):
    """base_decode_layer on the library's own scratch array (no workspace
    argument, nothing allocated); returns the filled base_plan (device
    pointers into that array)."""
    plan = base_plan() if plan is None else plan
    _check(load().base_decode_layer_noalloc(
        ctypes.byref(desc), _ptr(x), B, budget, flags, _ptr(residual), _ptr(y),
        ctypes.byref(plan), _stream(stream)))
    return plan


NOALLOC_SCRATCH_BYTES = 64 << 20


def base_pack_experts(desc, w13_packed, w2_packed, stream=None):
    _check(load().base_pack_experts(ctypes.byref(desc), _ptr(w13_packed),
                                    _ptr(w2_packed), _stream(stream)))


def packed_layer(layer: "Layer", K: int, stream=None) -> "Layer":
    """A Layer sharing router/predictor tensors, with expert weights packed
    into new tensors by base_pack_experts (one-time, on the device)."""
    import torch
    w_router, b_router, pred_a, pred_b, w13, w2 = layer.tensors
    w13p, w2p = torch.empty_like(w13), torch.empty_like(w2)
    base_pack_experts(layer.desc(K), w13p, w2p, stream)
    shared = None
    if layer.shared is not None:
        w13s, w2s, gate = layer.shared
        d = base_layer(layer.d, int(w13s.shape[0]), 1, layer.I, layer.dtype, layer.norm_topk,
                       W_ROWMAJOR, 0, None, None, None, None, _ptr(w13s), _ptr(w2s),
                       0, None, None, None)
        w13sp, w2sp = torch.empty_like(w13s), torch.empty_like(w2s)
        base_pack_experts(d, w13sp, w2sp, stream)
        shared = (w13sp, w2sp, gate)
    return Layer(w_router, b_router, pred_a, pred_b, w13p, w2p,
                 layer.norm_topk, W_PACKED, layer.score_rule, shared)


def base_set_stage_events(events):
    """events: a sequence of 2 * N_STAGES raw hipEvent_t handles (start and
    end of each stage's kernel), or None."""
    if events is None:
        _check(load().base_set_stage_events(None, 0))
        return None
    arr = (ctypes.c_void_p * len(events))(*events)
    _check(load().base_set_stage_events(arr, len(events)))
    return arr   # keep alive while timing is on


def layer_stages(desc, B, budget):
    """Names of the stages base_decode_layer launches a kernel for."""
    m = _i32()
    _check(load().base_layer_stages(ctypes.byref(desc), B, budget, ctypes.byref(m)))
    return tuple(s for i, s in enumerate(STAGES) if m.value >> i & 1)


# App. A: the ridge's lambdas, 25 values log-spaced over [1e-4, 1e2]
CALIB_LAMBDAS = tuple(10.0 ** (-4.0 + 6.0 * i / 24) for i in range(25))


def calib_stats(desc: base_layer):
    """A zeroed statistics buffer (torch uint8 tensor on the device)."""
    import torch
    n = int(load().base_calib_stats_bytes(ctypes.byref(desc)))
    if n == 0:
        raise BaseError(-2, "shape outside the supported limits")
    stats = torch.empty(n, dtype=torch.uint8, device="cuda")
    _check(load().base_calib_reset(ctypes.byref(desc), _ptr(stats), _stream(None)))
    return stats


def calib_accumulate(desc, z, B, stats, ws=None, stream=None):
    """Adds one batch of calibration hidden states z [B, d] to stats."""
    import torch
    if ws is None:
        ws = torch.empty(int(load().base_calib_ws_bytes(ctypes.byref(desc), B)),
                         dtype=torch.uint8, device="cuda")
    _check(load().base_calib_accumulate(ctypes.byref(desc), _ptr(z), B, _ptr(stats),
                                        _ptr(ws), ws.numel(), _stream(stream)))
    return ws


def calib_fit(desc, stats, lambdas, pred_a, pred_b, lam_out=None, stream=None):
    """pred_a [E, d], pred_b [E] (fp32 device tensors) from the statistics;
    lambdas: a sequence of positive floats (host)."""
    lam = (ctypes.c_double * len(lambdas))(*[float(v) for v in lambdas])
    _check(load_calib().base_calib_fit(ctypes.byref(desc), _ptr(stats), len(lambdas), lam,
                                       _ptr(pred_a), _ptr(pred_b), _ptr(lam_out),
                                       _stream(stream)))


def plan_offset(plan: base_plan, field: str, ws) -> int:
    """Byte offset of a plan array inside the workspace tensor."""
    p = getattr(plan, field)
    return None if p is None else p - ws.data_ptr()
