"""Python binding of libstar (ctypes; argument marshalling only).

Every function here forwards torch tensors' device pointers and the current
HIP stream to the C-ABI entry point of the same name in ``libstar.so``; all
arithmetic runs in the library's gfx950 kernels.  There is no fallback: if
the library is missing, importing the binding's entry points raises.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libstar.so")

STAR_OK = 0
STAR_ERR_DEVICE_INPUT = -6
STAR_ERR_SCRATCH_LIMIT = -7
STAR_NOALLOC_SCRATCH_BYTES = 32 << 20
STAR_ABI_VERSION = 2
STAR_WS_HEADER_BYTES = 8192
STAR_MAX_TOP_K = 1024
F32, BF16 = 0, 1
ACT_RELU, ACT_GELU = 0, 1
DEV_BAD_INST, DEV_BAD_CUR, DEV_BAD_REM = 1, 2, 4

_i32 = ctypes.c_int32
_P = ctypes.c_void_p


class PredictParams(ctypes.Structure):
    _fields_ = [("n_req", _i32), ("d_model", _i32), ("d_hidden", _i32), ("n_bins", _i32),
                ("dtype", _i32), ("act", _i32), ("ema_alpha", ctypes.c_float),
                ("ema_init", _i32), ("len_max", _i32)]


class Mlp4Params(ctypes.Structure):
    _fields_ = [("n_req", _i32), ("d_model", _i32), ("m1", _i32), ("m2", _i32), ("m3", _i32),
                ("dtype", _i32), ("ema_alpha", ctypes.c_float), ("ema_init", _i32),
                ("len_max", _i32), ("b4", ctypes.c_float)]


class LoadParams(ctypes.Structure):
    _fields_ = [("n_req", _i32), ("n_inst", _i32), ("bucket", _i32), ("n_buckets", _i32)]


class ScoreParams(ctypes.Structure):
    _fields_ = [("load", LoadParams), ("top_k", _i32)]


class PlanParams(ctypes.Structure):
    _fields_ = [("load", LoadParams), ("max_moves", _i32), ("theta_num", _i32),
                ("theta_den", _i32), ("u_rule", _i32), ("mem_rule", _i32), ("min_rem", _i32),
                ("mem_cap", ctypes.c_int64)]


class StarError(RuntimeError):
    def __init__(self, fn: str, status: int, msg: str):
        super().__init__(f"{fn}: {msg} ({status})")
        self.status = status


class StarLibraryMissing(RuntimeError):
    pass


_lib = None


def lib():
    """The loaded libstar.so (raises StarLibraryMissing if it was not built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise StarLibraryMissing(
                f"{LIB_PATH} is missing: build it with `python -m paper_2510_13668_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        L.star_abi_version.restype = _i32
        if L.star_abi_version() != STAR_ABI_VERSION:
            raise StarLibraryMissing(
                f"{LIB_PATH} has ABI version {L.star_abi_version()}, this binding needs "
                f"{STAR_ABI_VERSION}: rebuild it with `python -m paper_2510_13668_amd.build`")
        L.star_status_string.restype = ctypes.c_char_p
        L.star_status_string.argtypes = [ctypes.c_int]
        L.star_predict_workspace_size.restype = ctypes.c_size_t
        L.star_predict_workspace_size.argtypes = [ctypes.POINTER(PredictParams)]
        L.star_project_load_workspace_size.restype = ctypes.c_size_t
        L.star_project_load_workspace_size.argtypes = [ctypes.POINTER(LoadParams)]
        L.star_score_workspace_size.restype = ctypes.c_size_t
        L.star_score_workspace_size.argtypes = [ctypes.POINTER(ScoreParams)]
        L.star_predict.restype = ctypes.c_int
        L.star_predict.argtypes = [ctypes.POINTER(PredictParams)] + [_P] * 10 + [ctypes.c_size_t, _P]
        L.star_predict_noalloc.argtypes = [ctypes.POINTER(PredictParams)] + [_P] * 10
        L.star_predict_overlap.argtypes = ([ctypes.POINTER(PredictParams)] + [_P] * 11 +
                                           [ctypes.c_size_t, _P])
        L.star_predict_overlap.restype = ctypes.c_int
        L.star_predict_overlap_workspace_size.argtypes = [ctypes.POINTER(PredictParams)]
        L.star_predict_overlap_workspace_size.restype = ctypes.c_size_t
        L.star_project_load.restype = ctypes.c_int
        L.star_project_load.argtypes = [ctypes.POINTER(LoadParams)] + [_P] * 5 + [ctypes.c_size_t, _P]
        L.star_score_migrations.restype = ctypes.c_int
        L.star_score_migrations.argtypes = ([ctypes.POINTER(ScoreParams)] + [_P] * 11 +
                                            [ctypes.c_size_t, _P])
        L.star_project_and_score_workspace_size.restype = ctypes.c_size_t
        L.star_project_and_score_workspace_size.argtypes = [ctypes.POINTER(ScoreParams)]
        L.star_project_and_score.restype = ctypes.c_int
        L.star_project_and_score.argtypes = ([ctypes.POINTER(ScoreParams)] + [_P] * 11 +
                                             [ctypes.c_size_t, _P])
        L.star_score_variance_workspace_size.restype = ctypes.c_size_t
        L.star_score_variance_workspace_size.argtypes = [ctypes.POINTER(LoadParams)]
        L.star_score_variance.restype = ctypes.c_int
        L.star_score_variance.argtypes = ([ctypes.POINTER(LoadParams)] + [_P] * 10 +
                                          [ctypes.c_size_t, _P])
        L.star_plan_workspace_size.restype = ctypes.c_size_t
        L.star_plan_workspace_size.argtypes = [ctypes.POINTER(PlanParams)]
        L.star_plan_migrations.restype = ctypes.c_int
        L.star_plan_migrations.argtypes = ([ctypes.POINTER(PlanParams)] + [_P] * 8 +
                                           [ctypes.c_size_t, _P])
        L.star_predict_mlp4_workspace_size.restype = ctypes.c_size_t
        L.star_predict_mlp4_workspace_size.argtypes = [ctypes.POINTER(Mlp4Params)]
        L.star_predict_mlp4.restype = ctypes.c_int
        L.star_predict_mlp4.argtypes = ([ctypes.POINTER(Mlp4Params)] + [_P] * 12 +
                                        [ctypes.c_size_t, _P])
        L.star_workspace_init.restype = ctypes.c_int
        L.star_workspace_init.argtypes = [_P, ctypes.c_size_t, _P]
        L.star_read_device_error.restype = ctypes.c_int
        L.star_read_device_error.argtypes = [_P, _P, ctypes.POINTER(_i32)]
        _lib = L
    return _lib


def _check(fn: str, st: int):
    if st != STAR_OK:
        raise StarError(fn, st, lib().star_status_string(st).decode())


def _ptrs(*ts):
    """Device addresses of contiguous device tensors (None stays None).

    One pass of cheap attribute reads, plain integers for ctypes and the raw
    current stream (below): one star_predict call went from 13.7 to 9.9 us of
    host time, which back-to-back calls on small batches wait for.
    """
    out = []
    for t in ts:
        if t is None:
            out.append(None)
            continue
        if not t.is_cuda:
            raise ValueError("libstar takes device tensors")
        if not t.is_contiguous():
            raise ValueError("tensors passed to libstar must be contiguous")
        out.append(t.data_ptr())
    return out


def _ptr(t: Optional[torch.Tensor]):
    """The address of one tensor (see _ptrs)."""
    return _ptrs(t)[0]


# torch's own shortcut past a Stream object (0.3 against 2.7 us of host time a call);
# not part of its documented interface, so a release without it takes the
# documented way
_raw_current_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream(stream) -> int:
    """The hipStream_t of `stream`, or of the current device's current stream."""
    if stream is None:
        if _raw_current_stream is not None:
            return _raw_current_stream(torch.cuda.current_device())
        stream = torch.cuda.current_stream()
    return stream.cuda_stream


# ---------------------------------------------------------------------------
# workspace
# ---------------------------------------------------------------------------
class Workspace:
    """Caller-owned device workspace (header zeroed on creation)."""

    def __init__(self, nbytes: int, device=None, stream=None):
        nbytes = max(int(nbytes), STAR_WS_HEADER_BYTES)
        self.buf = torch.empty(nbytes + 256, dtype=torch.uint8, device=device or "cuda")
        off = (-self.buf.data_ptr()) % 256
        self.ptr = self.buf.data_ptr() + off
        self.nbytes = nbytes
        _check("star_workspace_init", lib().star_workspace_init(self.ptr,
                                                                 self.nbytes, _stream(stream)))

    def read_device_error(self, stream=None) -> int:
        """The device-error word (0 = clean); STAR_ERR_DEVICE_INPUT is its
        non-zero status, not a failure of the call."""
        code = _i32(0)
        st = lib().star_read_device_error(self.ptr, _stream(stream),
                                          ctypes.byref(code))
        if st != STAR_ERR_DEVICE_INPUT:
            _check("star_read_device_error", st)
        return code.value


# ---------------------------------------------------------------------------
# (a) predictor
# ---------------------------------------------------------------------------
def predict_params(n_req, d_model, d_hidden, n_bins, dtype, act, ema_alpha=0.0, ema_init=False,
                   len_max=1 << 30) -> PredictParams:
    return PredictParams(n_req, d_model, d_hidden, n_bins, dtype, act, float(ema_alpha),
                         int(bool(ema_init)), int(len_max))


def predict_workspace_size(p: PredictParams) -> int:
    return lib().star_predict_workspace_size(ctypes.byref(p))


def predict(p: PredictParams, hidden, w1, b1, w2, b2, bin_values, ema_state, expected_len,
            rem_len, ws: Workspace, stream=None):
    _check("star_predict", lib().star_predict(
        ctypes.byref(p), *_ptrs(hidden, w1, b1, w2, b2, bin_values, ema_state, expected_len,
                                rem_len),
        ws.ptr, ws.nbytes, _stream(stream)))


def predict_noalloc(p: PredictParams, hidden, w1, b1, w2, b2, bin_values, ema_state,
                    expected_len, rem_len, stream=None):
    """star_predict without a workspace (the library's fixed device scratch)."""
    _check("star_predict_noalloc", lib().star_predict_noalloc(
        ctypes.byref(p), *_ptrs(hidden, w1, b1, w2, b2, bin_values, ema_state, expected_len,
                                rem_len),
        _stream(stream)))


def predict_overlap_workspace_size(p: PredictParams) -> int:
    return lib().star_predict_overlap_workspace_size(ctypes.byref(p))


def predict_overlap(p: PredictParams, hidden_next, ws_next, ws_prev, w1, b1, w2, b2,
                    bin_values, ema_state, expected_len, rem_len, stream=None):
    """star_predict_overlap: the head of the batch whose product `ws_prev`
    holds (None: no head) and the product of `hidden_next` into `ws_next`
    (None: no product), in one launch where the plan allows."""
    nbytes = (ws_next or ws_prev).nbytes
    _check("star_predict_overlap", lib().star_predict_overlap(
        ctypes.byref(p), _ptr(hidden_next), ws_next.ptr if ws_next else None,
        ws_prev.ptr if ws_prev else None,
        *_ptrs(w1, b1, w2, b2, bin_values, ema_state, expected_len, rem_len), nbytes,
        _stream(stream)))


# ---------------------------------------------------------------------------
# (b) load projection
# ---------------------------------------------------------------------------
def load_params(n_req, n_inst, bucket, n_buckets) -> LoadParams:
    return LoadParams(n_req, n_inst, bucket, n_buckets)


def project_load_workspace_size(p: LoadParams) -> int:
    return lib().star_project_load_workspace_size(ctypes.byref(p))


def project_load(p: LoadParams, cur_len, rem_len, inst_of, load, ws: Workspace, stream=None):
    _check("star_project_load", lib().star_project_load(
        ctypes.byref(p), *_ptrs(cur_len, rem_len, inst_of, load),
        ws.ptr, ws.nbytes, _stream(stream)))


# ---------------------------------------------------------------------------
# (c) scoring and ranking
# ---------------------------------------------------------------------------
def score_params(n_req, n_inst, bucket, n_buckets, top_k) -> ScoreParams:
    return ScoreParams(LoadParams(n_req, n_inst, bucket, n_buckets), top_k)


def score_workspace_size(p: ScoreParams) -> int:
    return lib().star_score_workspace_size(ctypes.byref(p))


def score_migrations(p: ScoreParams, cur_len, rem_len, inst_of, load, scores, best_target,
                     best_score, topk_req, topk_tgt, topk_score, ws: Workspace, stream=None):
    _check("star_score_migrations", lib().star_score_migrations(
        ctypes.byref(p), *_ptrs(cur_len, rem_len, inst_of, load, scores, best_target, best_score,
                                topk_req, topk_tgt, topk_score),
        ws.ptr, ws.nbytes, _stream(stream)))


def project_and_score_workspace_size(p: ScoreParams) -> int:
    return lib().star_project_and_score_workspace_size(ctypes.byref(p))


def project_and_score(p: ScoreParams, cur_len, rem_len, inst_of, load, scores, best_target,
                      best_score, topk_req, topk_tgt, topk_score, ws: Workspace, stream=None):
    """star_project_and_score: load projection and migration scoring in one
    call (`load` is an output)."""
    _check("star_project_and_score", lib().star_project_and_score(
        ctypes.byref(p), *_ptrs(cur_len, rem_len, inst_of, load, scores, best_target, best_score,
                                topk_req, topk_tgt, topk_score),
        ws.ptr, ws.nbytes, _stream(stream)))


# ---------------------------------------------------------------------------
# time-weighted variance gains
# ---------------------------------------------------------------------------
MOVE_FIELDS = 8   # star_move as int32 words: req, src, tgt, reserved, gain (4 words)


def score_variance_workspace_size(p: LoadParams) -> int:
    return int(lib().star_score_variance_workspace_size(ctypes.byref(p)))


def score_variance(p: LoadParams, cur_len, rem_len, inst_of, load, beta, gain, best_target,
                   best_gain, best_move, ws: Workspace, stream=None):
    """star_score_variance.  128-bit outputs are int64 tensors with a trailing
    dimension of 2 (low word, high word): gain [N, n, 2], best_gain [N, 2];
    best_move is an int32 tensor of MOVE_FIELDS words.  beta is int16 bits of
    the uint16 weights [K]."""
    _check("star_score_variance", lib().star_score_variance(
        ctypes.byref(p), *_ptrs(cur_len, rem_len, inst_of, load, beta, gain, best_target,
                                best_gain, best_move),
        ws.ptr, ws.nbytes, _stream(stream)))


def i128_to_int(lo: int, hi: int) -> int:
    """One (low, high) int64 pair of a 128-bit two's complement value."""
    return (int(hi) << 64) + (int(lo) & ((1 << 64) - 1))


# ---------------------------------------------------------------------------
# migration plans (Algorithm 1 end to end)
# ---------------------------------------------------------------------------
def plan_params(n_req, n_inst, bucket, n_buckets, max_moves, theta=(0, 1), u_rule=0,
                mem_rule=0, min_rem=0, mem_cap=(1 << 62)) -> PlanParams:
    return PlanParams(load_params(n_req, n_inst, bucket, n_buckets), max_moves, theta[0],
                      theta[1], u_rule, mem_rule, min_rem, mem_cap)


def plan_workspace_size(p: PlanParams) -> int:
    return int(lib().star_plan_workspace_size(ctypes.byref(p)))


def plan_migrations(p: PlanParams, cur_len, rem_len, inst_of, load, beta, moves, n_moves,
                    ws: Workspace, stream=None):
    """star_plan_migrations: inst_of and load are updated in place; moves is
    an int32 tensor of max_moves * MOVE_FIELDS words, n_moves int32 [1]."""
    _check("star_plan_migrations", lib().star_plan_migrations(
        ctypes.byref(p), *_ptrs(cur_len, rem_len, inst_of, load, beta, moves, n_moves),
        ws.ptr, ws.nbytes, _stream(stream)))


# ---------------------------------------------------------------------------
# the paper's regression head
# ---------------------------------------------------------------------------
def mlp4_params(n_req, d_model, m1, m2, m3, dtype, ema_alpha=0.0, ema_init=False,
                len_max=1 << 30, b4=0.0) -> Mlp4Params:
    return Mlp4Params(n_req, d_model, m1, m2, m3, dtype, ema_alpha, int(bool(ema_init)), len_max,
                      b4)


def predict_mlp4_workspace_size(p: Mlp4Params) -> int:
    return int(lib().star_predict_mlp4_workspace_size(ctypes.byref(p)))


def predict_mlp4(p: Mlp4Params, hidden, w1, b1, w2, b2, w3, b3, w4, ema_state, expected_len,
                 rem_len, ws: Workspace, stream=None):
    _check("star_predict_mlp4", lib().star_predict_mlp4(
        ctypes.byref(p), *_ptrs(hidden, w1, b1, w2, b2, w3, b3, w4, ema_state, expected_len,
                                rem_len),
        ws.ptr,
        ws.nbytes, _stream(stream)))
