"""Python binding of libhedgespec.so, the MI355X drafter-evaluation hot path of HedgeSpec.

Argument marshalling only: every step runs in the library's HIP kernels. PyTorch supplies
device memory and the current HIP stream. The function names match the C ABI declared in
include/hedgespec.h (hs_softmax_stats, hs_eval_alpha, hs_eval_topl, hs_accept_len,
hs_hedge_update, hs_normalhedge_update, hs_delayed_update, hs_play, hs_regret_update,
hs_round). There is no CPU fallback: if the library is not built,
loading raises.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# HS_LIBRARY: another build of the library to load (e.g. one with host sanitizers)
LIB_PATH = os.environ.get("HS_LIBRARY") or os.path.join(_HERE, "libhedgespec.so")

HS_OK = 0
HS_F32, HS_BF16, HS_F16 = 0, 1, 2
SAMPLE, GREEDY = 0, 1
LOSS_LENGTH, LOSS_ACCEPT_TOKEN, LOSS_ACCEPT_CHUNK = 0, 1, 2
MAX_DRAFTERS = 64
MAX_POSITIONS = 64
MAX_TOPL = 32  # HS_MAX_TOPL


class HsError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__("%s: %s" % (_status_name(code), msg))
        self.code = code


class hs_view(ctypes.Structure):
    _fields_ = [("ptr", ctypes.c_void_p), ("stride_b", ctypes.c_int64),
                ("stride_k", ctypes.c_int64)]


class hs_round_args(ctypes.Structure):
    _fields_ = [
        ("target", hs_view), ("drafters_host", ctypes.POINTER(hs_view)),
        ("N", ctypes.c_int), ("B", ctypes.c_int), ("K", ctypes.c_int), ("V", ctypes.c_int64),
        ("dtype", ctypes.c_int), ("temperature", ctypes.c_float), ("mode", ctypes.c_int),
        ("alpha", ctypes.c_void_p), ("agree", ctypes.c_void_p), ("argmax_t", ctypes.c_void_p),
        ("argmax_d", ctypes.c_void_p), ("parent_host", ctypes.c_void_p),
        ("path_end", ctypes.c_void_p), ("eal", ctypes.c_void_p), ("prefix", ctypes.c_void_p),
        ("loss_kind", ctypes.c_int), ("loss", ctypes.c_void_p), ("logw", ctypes.c_void_p),
        ("w", ctypes.c_void_p), ("eta", ctypes.c_double), ("R", ctypes.c_void_p),
        ("p", ctypes.c_void_p), ("c", ctypes.c_void_p), ("workspace", ctypes.c_void_p),
        ("workspace_bytes", ctypes.c_size_t),
    ]


_lib = None


def load_library(path: str = LIB_PATH) -> ctypes.CDLL:
    """Load libhedgespec.so (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(path):
        raise RuntimeError("libhedgespec.so is not built (%s); run __graft_entry__.build() or "
                           "python -m paper_2510_20064_amd.build" % path)
    lib = ctypes.CDLL(path)
    P, I, I64, F, D, SZ = (ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_float,
                           ctypes.c_double, ctypes.c_size_t)
    VP = ctypes.POINTER(hs_view)
    lib.hs_softmax_stats.argtypes = [P, I, I64, I64, I64, F, P, P, P, P]
    lib.hs_eval_alpha_workspace_size.argtypes = [I, I, I, I64, I]
    lib.hs_eval_alpha_workspace_size.restype = SZ
    lib.hs_eval_alpha.argtypes = [VP, VP, I, I, I, I64, I, F, I, P, P, P, P, P, SZ, P]
    lib.hs_eval_alpha_noalloc.argtypes = [VP, VP, I, I, I, I64, I, F, I, P, P, P, P, P]
    lib.hs_eval_alpha_noalloc_max_workspace.argtypes = []
    lib.hs_eval_alpha_noalloc_max_workspace.restype = SZ
    lib.hs_eval_topl_workspace_size.argtypes = [I, I, I, I64, I, I]
    lib.hs_eval_topl_workspace_size.restype = SZ
    lib.hs_eval_topl.argtypes = [VP, VP, I, I, I, I64, I, I, F, I, P, P, P, P, SZ, P]
    lib.hs_candidate_mass.argtypes = [VP, I, I, I, I64, I, F, P, P, I, P, P]
    lib.hs_play.argtypes = [P, I, I, I, P, P, P]
    lib.hs_regret_update.argtypes = [P, I, I, I, P, P, P, P, P, P, P]
    lib.hs_accept_len.argtypes = [P, P, I, I, I, I, P, P, P, P, I, P, P]
    lib.hs_hedge_update.argtypes = [P, P, P, I, I, I, D, P]
    lib.hs_normalhedge_update.argtypes = [P, P, P, P, I, I, I, P]
    lib.hs_round.argtypes = [ctypes.POINTER(hs_round_args), P]
    lib.hs_delayed_update.argtypes = [P, P, I, I, I, I, P, I64, P, P, P, P, D, P, P, P, P, P, P]
    lib.hs_set_wait_limit.argtypes = [I]
    lib.hs_set_wait_limit.restype = None
    lib.hs_stream_read.argtypes = [P, SZ, I, I, I, P, P]
    lib.hs_status_string.argtypes = [I]
    lib.hs_status_string.restype = ctypes.c_char_p
    lib.hs_last_error.restype = ctypes.c_char_p
    for name in ["hs_softmax_stats", "hs_eval_alpha", "hs_eval_alpha_noalloc", "hs_eval_topl", "hs_play", "hs_regret_update",
                 "hs_accept_len", "hs_hedge_update",
                 "hs_normalhedge_update", "hs_round", "hs_delayed_update", "hs_version"]:
        getattr(lib, name).restype = I
    _lib = lib
    return lib


def _status_name(code: int) -> str:
    try:
        return load_library().hs_status_string(code).decode()
    except Exception:  # pragma: no cover
        return "status %d" % code


def _check(code: int) -> None:
    if code != HS_OK:
        raise HsError(code, load_library().hs_last_error().decode())


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream(stream=None):
    s = torch.cuda.current_stream() if stream is None else stream
    return ctypes.c_void_p(s.cuda_stream)


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return HS_F32
    if t.dtype in (torch.bfloat16, torch.uint16, torch.int16):
        return HS_BF16
    if t.dtype == torch.float16:
        return HS_F16
    raise TypeError("logits must be float32, bfloat16 or float16, got %s" % t.dtype)


def _view(t: torch.Tensor) -> hs_view:
    if t.dim() != 3 or t.stride(2) != 1:
        raise ValueError("a logits view must be [B][K][V] with V contiguous")
    return hs_view(t.data_ptr(), t.stride(0), t.stride(1))


# --------------------------------------------------------------------------------------------

def softmax_stats(x: torch.Tensor, V: Optional[int] = None, temperature: float = 1.0,
                  stream=None, out=None):
    """hs_softmax_stats on a [rows][ld] tensor: returns (row_max f32, row_lse f32, row_argmax i32),
    written into `out` (the same three tensors) when it is given."""
    lib = load_library()
    rows, ld = x.shape
    V = ld if V is None else V
    if x.stride(1) != 1:
        raise ValueError("rows must be contiguous")
    if out is None:
        mx = torch.empty(rows, dtype=torch.float32, device=x.device)
        lse = torch.empty(rows, dtype=torch.float32, device=x.device)
        am = torch.empty(rows, dtype=torch.int32, device=x.device)
    else:
        mx, lse, am = out
        for o, dt in ((mx, torch.float32), (lse, torch.float32), (am, torch.int32)):
            if o.dtype != dt or o.numel() != rows or not o.is_contiguous() or o.device != x.device:
                raise ValueError("out: three contiguous [rows] tensors (f32, f32, i32) on x's device")
    _check(lib.hs_softmax_stats(_ptr(x), _dtype_code(x), rows, V, x.stride(0), temperature,
                                _ptr(mx), _ptr(lse), _ptr(am), _stream(stream)))
    return mx, lse, am


def set_wait_limit(polls: int) -> None:
    """hs_set_wait_limit: polls before a wait inside the evaluation kernel gives up (negative:
    the default; 0: every wait gives up at once, to exercise the failure path)."""
    load_library().hs_set_wait_limit(int(polls))


def stream_read(x: torch.Tensor, grid: int = 2048, unroll: int = 4, nontemporal: bool = False,
                out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """hs_stream_read: read every byte of the contiguous device tensor x once (a measurement
    aid: the device's streaming read rate); returns the grid * 4 per-wave XOR words."""
    if not x.is_contiguous():
        raise ValueError("x must be contiguous")
    if out is None:
        out = torch.empty(grid * 4, dtype=torch.int32, device=x.device)
    elif out.numel() < grid * 4 or out.dtype != torch.int32 or out.device != x.device:
        raise ValueError("out: at least grid * 4 int32 words on x's device")
    _check(load_library().hs_stream_read(_ptr(x), x.numel() * x.element_size(), grid, unroll,
                                         int(bool(nontemporal)), _ptr(out), _stream(stream)))
    return out


def eval_workspace_size(B: int, N: int, K: int, V: int, dtype: int) -> int:
    return int(load_library().hs_eval_alpha_workspace_size(B, N, K, V, dtype))


def alloc_workspace(B: int, N: int, K: int, V: int, dtype: int, device) -> torch.Tensor:
    n = eval_workspace_size(B, N, K, V, dtype)
    if n == 0:
        raise ValueError("invalid shape for the evaluation workspace")
    # zero-filled once; every completed call leaves it zero-filled again
    return torch.zeros(n, dtype=torch.uint8, device=device)


def _split_logits(target: torch.Tensor, drafters):
    """Accept a [N+1][B][K][V] tensor (row 0 target) or (target [B][K][V], drafters list/tensor)."""
    if drafters is None:
        return target[0], [target[1 + i] for i in range(target.shape[0] - 1)]
    if isinstance(drafters, torch.Tensor):
        return target, [drafters[i] for i in range(drafters.shape[0])]
    return target, list(drafters)


def _logit_views(target: torch.Tensor, drafters):
    """The C views of _split_logits: (target, drafters, N, B, K, row length). A stack of drafters is
    addressed from its base and strides instead of one tensor slice per drafter, which the host
    took longer for than the GPU for the call: a top-L call for one query and 8 drafters 27.9 us, of
    which the kernels need 16, and 19.0 us so."""
    stack = target if drafters is None else drafters
    if (isinstance(stack, torch.Tensor) and stack.dim() == 4 and stack.stride(3) == 1
            and stack.numel() > 0 and (drafters is None or target.dim() == 3)):
        n, B, K, ld = stack.shape
        s0, sb, sk, _ = stack.stride()
        step = s0 * stack.element_size()
        base = stack.data_ptr()
        rows = [hs_view(base + i * step, sb, sk) for i in range(n)]
        if drafters is None:
            return rows[0], (hs_view * (n - 1))(*rows[1:]), n - 1, B, K, ld
        B, K, ld = target.shape
        return _view(target), (hs_view * n)(*rows), n, B, K, ld
    t, ds = _split_logits(target, drafters)
    B, K, ld = t.shape
    return _view(t), (hs_view * len(ds))(*[_view(d) for d in ds]), len(ds), B, K, ld


def eval_alpha(target: torch.Tensor, drafters=None, V: Optional[int] = None,
               temperature: float = 1.0, mode: int = SAMPLE, want_alpha: Optional[bool] = None,
               want_agree: Optional[bool] = None, want_argmax: bool = False,
               workspace: Optional[torch.Tensor] = None, out: Optional[dict] = None, stream=None):
    """hs_eval_alpha. Returns a dict of device tensors: alpha [B][N][K] f32, agree [B][N][K] u8,
    argmax_t [B][K] i32, argmax_d [B][N][K] i32 (those requested)."""
    lib = load_library()
    tv, dv, N, B, K, ld = _logit_views(target, drafters)
    V = ld if V is None else V
    dt = _dtype_code(target)
    dev = target.device
    want_alpha = (mode == SAMPLE) if want_alpha is None else want_alpha
    want_agree = (mode == GREEDY) if want_agree is None else want_agree
    o = {} if out is None else out
    if want_alpha and "alpha" not in o:
        o["alpha"] = torch.empty((B, N, K), dtype=torch.float32, device=dev)
    if want_agree and "agree" not in o:
        o["agree"] = torch.empty((B, N, K), dtype=torch.uint8, device=dev)
    if want_argmax:
        o.setdefault("argmax_t", torch.empty((B, K), dtype=torch.int32, device=dev))
        o.setdefault("argmax_d", torch.empty((B, N, K), dtype=torch.int32, device=dev))
    if workspace is None:
        workspace = alloc_workspace(B, N, K, V, dt, dev)
    _check(lib.hs_eval_alpha(ctypes.byref(tv), dv, N, B, K, V, dt, temperature, mode,
                             _ptr(o.get("alpha")), _ptr(o.get("agree")), _ptr(o.get("argmax_t")),
                             _ptr(o.get("argmax_d")), _ptr(workspace), workspace.numel(),
                             _stream(stream)))
    return o


def eval_alpha_noalloc(target: torch.Tensor, drafters=None, V: Optional[int] = None,
                       temperature: float = 1.0, mode: int = SAMPLE, out: Optional[dict] = None,
                       stream=None):
    """hs_eval_alpha_noalloc: hs_eval_alpha with the library's fixed workspace array instead of
    a caller's workspace. `out` holds preallocated outputs (alpha, agree, argmax_t, argmax_d;
    those present are filled); nothing is allocated when it covers what the mode requires."""
    lib = load_library()
    tv, dv, N, B, K, ld = _logit_views(target, drafters)
    V = ld if V is None else V
    o = {} if out is None else out
    if mode == SAMPLE and "alpha" not in o:
        o["alpha"] = torch.empty((B, N, K), dtype=torch.float32, device=target.device)
    if mode == GREEDY and "agree" not in o:
        o["agree"] = torch.empty((B, N, K), dtype=torch.uint8, device=target.device)
    _check(lib.hs_eval_alpha_noalloc(ctypes.byref(tv), dv, N, B, K, V, _dtype_code(target),
                                     temperature, mode, _ptr(o.get("alpha")), _ptr(o.get("agree")),
                                     _ptr(o.get("argmax_t")), _ptr(o.get("argmax_d")),
                                     _stream(stream)))
    return o


def candidate_mass(target: torch.Tensor, lse: torch.Tensor, cand: torch.Tensor,
                   V: Optional[int] = None, temperature: float = 1.0,
                   out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """hs_candidate_mass (Theorem 2 with dynamic pruning): the target's mass on given candidate
    sets. target [B][K][ld] logits, lse [B][K] f32 (natural-log normalisers at `temperature`,
    e.g. softmax_stats' row_lse), cand [B][N][K][C] i32 (negative = empty slot).
    Returns gamma [B][N][K] f32."""
    lib = load_library()
    B, K, ld = target.shape
    V = ld if V is None else V
    Bc, N, Kc, C = cand.shape
    if (Bc, Kc) != (B, K) or cand.dtype != torch.int32 or not cand.is_contiguous():
        raise ValueError("cand must be a contiguous int32 [B][N][K][C] tensor")
    if lse.shape != (B, K) or lse.dtype != torch.float32 or not lse.is_contiguous():
        raise ValueError("lse must be a contiguous float32 [B][K] tensor")
    if out is None:
        out = torch.empty((B, N, K), dtype=torch.float32, device=target.device)
    elif out.shape != (B, N, K) or out.dtype != torch.float32 or not out.is_contiguous():
        raise ValueError("out must be a contiguous float32 [B][N][K] tensor")
    tv = _view(target)
    _check(lib.hs_candidate_mass(ctypes.byref(tv), N, B, K, V, _dtype_code(target), temperature,
                                 _ptr(lse), _ptr(cand), C, _ptr(out), _stream(stream)))
    return out


def topl_workspace_size(B: int, N: int, K: int, V: int, L: int, dtype: int) -> int:
    return int(load_library().hs_eval_topl_workspace_size(B, N, K, V, L, dtype))


def eval_topl(target: torch.Tensor, drafters=None, L: int = 10, V: Optional[int] = None,
              temperature: float = 1.0, mode: int = SAMPLE, want_gamma: Optional[bool] = None,
              want_hit: Optional[bool] = None, want_children: bool = False,
              workspace: Optional[torch.Tensor] = None, out: Optional[dict] = None, stream=None):
    """hs_eval_topl (Theorem 2). Returns a dict of device tensors: gamma [B][N][K] f32,
    hit [B][N][K] u8, children [B][N][K][L] i32 (those requested)."""
    lib = load_library()
    tv, dv, N, B, K, ld = _logit_views(target, drafters)
    V = ld if V is None else V
    dt = _dtype_code(target)
    dev = target.device
    want_gamma = (mode == SAMPLE) if want_gamma is None else want_gamma
    want_hit = (mode == GREEDY) if want_hit is None else want_hit
    o = {} if out is None else out
    if want_gamma and "gamma" not in o:
        o["gamma"] = torch.empty((B, N, K), dtype=torch.float32, device=dev)
    if want_hit and "hit" not in o:
        o["hit"] = torch.empty((B, N, K), dtype=torch.uint8, device=dev)
    if want_children and "children" not in o:
        o["children"] = torch.empty((B, N, K, L), dtype=torch.int32, device=dev)
    if workspace is None:
        n = topl_workspace_size(B, N, K, V, L, dt)
        workspace = torch.empty(max(n, 1), dtype=torch.uint8, device=dev)
    _check(lib.hs_eval_topl(ctypes.byref(tv), dv, N, B, K, V, dt, L, temperature, mode,
                            _ptr(o.get("gamma")), _ptr(o.get("hit")), _ptr(o.get("children")),
                            _ptr(workspace), workspace.numel(), _stream(stream)))
    return o


def _parent_host(parent):
    if parent is None:
        return None, None
    arr = (ctypes.c_int32 * len(parent))(*[int(x) for x in parent])
    return arr, ctypes.cast(arr, ctypes.c_void_p)


def accept_len(gamma: torch.Tensor, mode: int = SAMPLE, parent: Optional[Sequence[int]] = None,
               path_end: Optional[torch.Tensor] = None, loss_kind: int = LOSS_LENGTH,
               want_prefix: bool = False, want_loss: bool = True, stream=None):
    """hs_accept_len. gamma: alpha [B][N][K] f32 (SAMPLE) or agree [B][N][K] u8 (GREEDY)."""
    lib = load_library()
    B, N, K = gamma.shape
    dev = gamma.device
    eal = torch.empty((B, N), dtype=torch.float64, device=dev)
    prefix = torch.empty((B, N, K), dtype=torch.float64, device=dev) if want_prefix else None
    L = K if loss_kind == LOSS_ACCEPT_TOKEN else 1
    loss = torch.empty((L, B, N), dtype=torch.float64, device=dev) if want_loss else None
    keep, par = _parent_host(parent)
    alpha = gamma if mode == SAMPLE else None
    agree = gamma if mode == GREEDY else None
    _check(lib.hs_accept_len(_ptr(alpha), _ptr(agree), mode, B, N, K, par, _ptr(path_end),
                             _ptr(eal), _ptr(prefix), loss_kind, _ptr(loss), _stream(stream)))
    del keep
    return {"eal": eal, "prefix": prefix, "loss": loss}


def hedge_update(logw: torch.Tensor, w: torch.Tensor, loss: torch.Tensor, eta: float,
                 stream=None) -> None:
    """hs_hedge_update in place: logw [B][N] in/out, w [B][N] out, loss [L][B][N]."""
    L, B, N = loss.shape
    _check(load_library().hs_hedge_update(_ptr(logw), _ptr(w), _ptr(loss), L, B, N, eta,
                                          _stream(stream)))


def normalhedge_update(R: torch.Tensor, p: torch.Tensor, c: torch.Tensor, loss: torch.Tensor,
                       stream=None) -> None:
    """hs_normalhedge_update in place: R, p [B][N] in/out, c [B] out, loss [L][B][N]."""
    L, B, N = loss.shape
    _check(load_library().hs_normalhedge_update(_ptr(R), _ptr(p), _ptr(c), _ptr(loss), L, B, N,
                                                _stream(stream)))


class LearnerState:
    """Device-resident per-query learner state: Hedge (logw, w) and NormalHedge (R, p, c)."""

    def __init__(self, B: int, N: int, device):
        self.logw = torch.zeros((B, N), dtype=torch.float64, device=device)
        self.w = torch.full((B, N), 1.0 / N, dtype=torch.float64, device=device)
        self.R = torch.zeros((B, N), dtype=torch.float64, device=device)
        self.p = torch.full((B, N), 1.0 / N, dtype=torch.float64, device=device)
        self.c = torch.zeros((B,), dtype=torch.float64, device=device)


class DelayedState:
    """Device state of hs_delayed_update for B queries, N drafters and window K: the feedback
    history ring, the per-query clock (tokens received, windows used) and the learners."""

    def __init__(self, B: int, N: int, K: int, device):
        self.B, self.N, self.K = B, N, K
        self.hist = torch.zeros((B, 2 * K, N), dtype=torch.float32, device=device)
        self.clock = torch.zeros((B, 2), dtype=torch.int64, device=device)
        self.learners = LearnerState(B, N, device)
        self.loss = torch.zeros((K, B, N), dtype=torch.float64, device=device)
        self.nloss = torch.zeros((B,), dtype=torch.int32, device=device)


def delayed_update(state: DelayedState, gamma: torch.Tensor, count: torch.Tensor, eta: float,
                   mode: int = SAMPLE, hedge: bool = True, normalhedge: bool = True,
                   hybrid_tokens: int = 0, stream=None) -> None:
    """hs_delayed_update: append query b's next count[b] tokens of feedback (gamma [B][N][K]:
    alpha fp32 in SAMPLE mode, agree uint8 in GREEDY mode) and feed every token loss that is
    now known (the K-token window's length loss; the acceptance loss for each query's first
    hybrid_tokens tokens) to the learners. The losses used are left in state.loss (first
    state.nloss[b] rows per query)."""
    B, N, K = gamma.shape
    st = state.learners
    alpha = gamma if mode == SAMPLE else None
    agree = gamma if mode == GREEDY else None
    _check(load_library().hs_delayed_update(
        _ptr(alpha), _ptr(agree), mode, B, N, K, _ptr(count), int(hybrid_tokens),
        _ptr(state.hist), _ptr(state.clock), _ptr(st.logw if hedge else None),
        _ptr(st.w if hedge else None), eta, _ptr(st.R if normalhedge else None),
        _ptr(st.p if normalhedge else None), _ptr(st.c if normalhedge else None),
        _ptr(state.loss), _ptr(state.nloss), _stream(stream)))


PLAY_ARGMAX, PLAY_SAMPLE = 0, 1


def play(weights: torch.Tensor, how: int = PLAY_ARGMAX, u: Optional[torch.Tensor] = None,
         out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """hs_play: the drafter each query plays, from weights [B][N] fp64 (argmax, or an
    inverse-CDF sample with the uniform draws u [B] fp64). Returns choice [B] int32."""
    B, N = weights.shape
    if out is None:
        out = torch.empty((B,), dtype=torch.int32, device=weights.device)
    _check(load_library().hs_play(_ptr(weights), B, N, how, _ptr(u), _ptr(out), _stream(stream)))
    return out


class RegretState:
    """Device regret bookkeeping for B queries and N drafters (hs_regret_update)."""

    def __init__(self, B: int, N: int, device):
        self.cum = torch.zeros((B, N), dtype=torch.float64, device=device)
        self.played = torch.zeros((B,), dtype=torch.float64, device=device)
        self.regret = torch.zeros((B,), dtype=torch.float64, device=device)
        self.eal_sum = torch.zeros((B,), dtype=torch.float64, device=device)

    def update(self, loss: torch.Tensor, played: torch.Tensor, eal: Optional[torch.Tensor] = None,
               stream=None) -> torch.Tensor:
        """loss [L][B][N] fp64, played [L][B] (or [B] for L = 1) int32."""
        L, B, N = loss.shape
        _check(load_library().hs_regret_update(
            _ptr(loss), L, B, N, _ptr(played), _ptr(self.cum), _ptr(self.played),
            _ptr(self.regret), _ptr(eal), _ptr(self.eal_sum if eal is not None else None),
            _stream(stream)))
        return self.regret


class UpdateCadence:
    """Batched delayed feedback (Appendix "Practical heuristics: skipping update"): the
    learners are updated every round during a warm-up, then only once every `batch` rounds,
    with all the feedback gathered since the last update. QFI-D applies the queued losses in
    token order either way, so after an update the learners hold exactly the state that
    per-round updates would give; only the predictions in between are older.

    push(gamma, count) keeps a device copy of the round's feedback (gamma [B][N][K], count [B])
    and, when the round is due, replays every kept round through hs_delayed_update in order.
    Returns whether the learners were updated. Scheduling only: the losses and the learner
    steps run in the library's kernel."""

    def __init__(self, state: DelayedState, eta: float, warmup: int = 6, batch: int = 12,
                 mode: int = SAMPLE, hybrid_tokens: int = 0):
        if warmup < 0 or batch < 1:
            raise ValueError("need warmup >= 0 and batch >= 1")
        self.state, self.eta, self.warmup, self.batch = state, eta, warmup, batch
        self.mode, self.hybrid_tokens = mode, hybrid_tokens
        self.rounds = 0
        self.pending = []

    def due(self, r: int) -> bool:
        """Whether round r (0-based) ends with an update of the learners."""
        return r < self.warmup or (r + 1 - self.warmup) % self.batch == 0

    def push(self, gamma: torch.Tensor, count: torch.Tensor, stream=None) -> bool:
        self.pending.append((gamma.clone(), count.clone()))
        r = self.rounds
        self.rounds += 1
        if not self.due(r):
            return False
        self.flush(stream)
        return True

    def flush(self, stream=None) -> None:
        for g, c in self.pending:
            delayed_update(self.state, g, c, self.eta, mode=self.mode,
                           hybrid_tokens=self.hybrid_tokens, stream=stream)
        self.pending = []


class Round:
    """Pre-marshalled hs_round call: eval + learner kernel for fixed buffers.

    Build once, then call run() per verification round (optionally switching the logits
    buffer with set_logits) - the ctypes structure is reused, so a call costs only the
    launches."""

    def __init__(self, target: torch.Tensor, drafters=None, V: Optional[int] = None,
                 temperature: float = 1.0, mode: int = SAMPLE, loss_kind: int = LOSS_LENGTH,
                 eta: float = 0.5, parent: Optional[Sequence[int]] = None,
                 path_end: Optional[torch.Tensor] = None, hedge: bool = True,
                 normalhedge: bool = True, want_prefix: bool = False, want_argmax: bool = False,
                 want_loss: bool = True, want_agree: Optional[bool] = None,
                 state: Optional[LearnerState] = None):
        self.lib = load_library()
        t, ds = _split_logits(target, drafters)
        B, K, ld = t.shape
        N = len(ds)
        self.B, self.N, self.K = B, N, K
        self.V = ld if V is None else V
        dev = t.device
        self.dtype = _dtype_code(t)
        self.mode = mode
        self.alpha = torch.empty((B, N, K), dtype=torch.float32, device=dev)
        self.agree = torch.empty((B, N, K), dtype=torch.uint8, device=dev)
        self.argmax_t = torch.empty((B, K), dtype=torch.int32, device=dev) if want_argmax else None
        self.argmax_d = (torch.empty((B, N, K), dtype=torch.int32, device=dev)
                         if want_argmax else None)
        self.eal = torch.empty((B, N), dtype=torch.float64, device=dev)
        self.prefix = torch.empty((B, N, K), dtype=torch.float64, device=dev) if want_prefix else None
        L = K if loss_kind == LOSS_ACCEPT_TOKEN else 1
        self.loss = torch.empty((L, B, N), dtype=torch.float64, device=dev) if want_loss else None
        self.state = state if state is not None else LearnerState(B, N, dev)
        self.workspace = alloc_workspace(B, N, K, self.V, self.dtype, dev)
        self._par_keep, par = _parent_host(parent)
        self.path_end = path_end
        self._views = (hs_view * N)()
        a = hs_round_args()
        a.drafters_host = ctypes.cast(self._views, ctypes.POINTER(hs_view))
        a.N, a.B, a.K, a.V = N, B, K, self.V
        a.dtype, a.temperature, a.mode = self.dtype, temperature, mode
        want_agree = (mode == GREEDY) if want_agree is None else want_agree
        a.alpha = self.alpha.data_ptr() if mode == SAMPLE else None
        a.agree = self.agree.data_ptr() if want_agree else None
        a.argmax_t = None if self.argmax_t is None else self.argmax_t.data_ptr()
        a.argmax_d = None if self.argmax_d is None else self.argmax_d.data_ptr()
        a.parent_host = par
        a.path_end = None if path_end is None else path_end.data_ptr()
        a.eal = self.eal.data_ptr()
        a.prefix = None if self.prefix is None else self.prefix.data_ptr()
        a.loss_kind = loss_kind
        a.loss = None if self.loss is None else self.loss.data_ptr()
        st = self.state
        if hedge:
            a.logw, a.w, a.eta = st.logw.data_ptr(), st.w.data_ptr(), eta
        if normalhedge:
            a.R, a.p, a.c = st.R.data_ptr(), st.p.data_ptr(), st.c.data_ptr()
        a.workspace = self.workspace.data_ptr()
        a.workspace_bytes = self.workspace.numel()
        self.args = a
        self.set_logits(target, drafters)

    def set_logits(self, target: torch.Tensor, drafters=None) -> None:
        t, ds = _split_logits(target, drafters)
        if len(ds) != self.N or tuple(t.shape[:2]) != (self.B, self.K):
            raise ValueError("logits shape changed")
        self._keep = (t, ds)
        self.args.target = _view(t)
        for i, d in enumerate(ds):
            self._views[i] = _view(d)

    def run(self, stream=None) -> None:
        _check(self.lib.hs_round(ctypes.byref(self.args), _stream(stream)))
