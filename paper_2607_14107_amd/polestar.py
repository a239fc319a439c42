"""Thin Python binding of libpolestar.so (the C ABI of include/polestar.h).

Argument marshalling only: tensors provide device memory (`data_ptr()`) and
the current HIP stream; every step of the computation runs in the library's
HIP kernels.  There is no CPU fallback: if the library is not built, or a
tensor is not on the GPU, the call raises.

Names follow the C entry points: drift, select, refresh_kv, attend, commit.
`Step` preallocates the buffers of one layer step and runs the five calls
back to back on one stream.
"""

from __future__ import annotations

import ctypes
import os

import torch

PKG = os.path.dirname(os.path.abspath(__file__))
# POLESTAR_LIB selects another build of the library (the host-sanitized one
# of the CPU tests); by default the in-tree libpolestar.so.
LIB_PATH = os.environ.get("POLESTAR_LIB") or os.path.join(PKG, "libpolestar.so")

OK = 0
STATUS = {0: "ok", 1: "invalid argument", 2: "unsupported", 3: "launch failed", 4: "workspace too small"}
FP32, BF16 = 0, 1
MXFP4, MXFP8 = 0, 1
CODECS = {"mxfp4": MXFP4, "mxfp8": MXFP8}

# hyperparameter defaults (table of default hyperparameters, App. D)
DEFAULT_TAU_S = 0.9
DEFAULT_ALPHA = 10.0
DEFAULT_HISTORY = 5

_lib = None


class PolestarError(RuntimeError):
    def __init__(self, fn: str, status: int):
        super().__init__(f"{fn}: {STATUS.get(status, status)} (status {status})")
        self.status = status


class StepArgs(ctypes.Structure):
    """Mirror of polestar_step_args (include/polestar.h), field for field."""
    _fields_ = [(n, ctypes.c_int) for n in (
        "dtype", "batch", "seq", "d", "n_heads", "n_kv_heads", "head_dim", "block_start", "block_len",
        "vocab", "k", "h", "mask_token_id", "force_one")] + \
        [(n, ctypes.c_float) for n in ("tau_s", "alpha", "scale")] + \
        [(n, ctypes.c_void_p) for n in (
            "h_cur", "h_prev", "eligible", "w_q", "w_k", "w_v", "k_cache", "v_cache", "logits", "masked",
            "hist", "hist_len", "drift", "stale_idx", "stale_count", "q", "out", "lse", "token", "conf",
            "commit")]


def lib() -> ctypes.CDLL:
    """Load libpolestar.so once and declare its signatures."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is not built: run paper_2607_14107_amd.build.build()")
    L = ctypes.CDLL(LIB_PATH)
    P, I, F, Z, S = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_size_t, ctypes.c_int
    L.polestar_version.restype = I
    L.polestar_version.argtypes = []
    L.polestar_status_string.restype = ctypes.c_char_p
    L.polestar_status_string.argtypes = [I]
    L.polestar_drift.restype = S
    L.polestar_drift.argtypes = [I, I, I, I, P, P, P, P]
    L.polestar_select.restype = S
    L.polestar_select.argtypes = [I, I, P, P, I, I, I, P, P, P]
    L.polestar_refresh_kv_workspace_size.restype = Z
    L.polestar_refresh_kv_workspace_size.argtypes = [I, I, I, I, I, I, I]
    L.polestar_refresh_kv.restype = S
    L.polestar_refresh_kv.argtypes = [I, I, I, I, I, I, P, P, P, I, I, I, P, P, P, P, P, Z, P]
    L.polestar_refresh_kv_noalloc_max_bytes.argtypes = []
    L.polestar_refresh_kv_noalloc_max_bytes.restype = Z
    L.polestar_refresh_kv_noalloc.argtypes = [I, I, I, I, I, I, P, P, P, I, I, I, P, P, P, P, P]
    L.polestar_refresh_kv_noalloc.restype = S
    L.polestar_project_qkv_workspace_size.restype = Z
    L.polestar_project_qkv_workspace_size.argtypes = [I, I, I, I, I, I, I]
    L.polestar_project_qkv.restype = S
    L.polestar_project_qkv.argtypes = [I, I, I, I, I, I, I, P, I, I, P, P, P, P, P, P, P, Z, P]
    L.polestar_project_q_workspace_size.restype = Z
    L.polestar_project_q_workspace_size.argtypes = [I, I, I, I, I, I]
    L.polestar_project_q.restype = S
    L.polestar_project_q.argtypes = [I, I, I, I, I, I, I, I, P, P, P, P, Z, P]
    L.polestar_attend_workspace_size.restype = Z
    L.polestar_attend_workspace_size.argtypes = [I, I, I, I, I, I, I, I]
    L.polestar_attend.restype = S
    L.polestar_attend.argtypes = [I, I, I, I, I, I, I, I, I, P, P, P, P, P, F, P, P, P, Z, P]
    L.polestar_cluster.restype = S
    L.polestar_cluster.argtypes = [I, I, I, I, P, P, I, I, I, P, P, P, P, P]
    L.polestar_proxy_drift_workspace_size.restype = Z
    L.polestar_proxy_drift_workspace_size.argtypes = [I, I, I, I, I, I, I]
    L.polestar_proxy_drift.restype = S
    L.polestar_proxy_drift.argtypes = [I, I, I, I, I, I, I, I, P, P, P, P, F, P, P, I, P, P, Z, P]
    L.polestar_cluster_select.restype = S
    L.polestar_cluster_select.argtypes = [I, I, P, I, P, I, P, I, P, P]
    L.polestar_cluster_update.restype = S
    L.polestar_cluster_update.argtypes = [I, I, I, I, P, P, P, I, P, P, I, P, P]
    L.polestar_step_workspace_size.restype = Z
    L.polestar_step_workspace_size.argtypes = [ctypes.POINTER(StepArgs)]
    L.polestar_step.restype = S
    L.polestar_step.argtypes = [ctypes.POINTER(StepArgs), P, Z, P, P, P]
    L.polestar_commit_workspace_size.restype = Z
    L.polestar_commit_workspace_size.argtypes = [I, I, I, I]
    L.polestar_commit.restype = S
    L.polestar_commit.argtypes = [I, I, I, I, P, P, P, I, I, P, P, I, I, F, F, I, P, P, P, P, Z, P]
    L.polestar_suffix_commit.restype = S
    L.polestar_suffix_commit.argtypes = [I, I, I, I, P, P, P, I, F, P, P, P, P, Z, P]
    L.polestar_attention_drift_workspace_size.restype = Z
    L.polestar_attention_drift_workspace_size.argtypes = [I, I, I, I]
    L.polestar_attention_drift.restype = S
    L.polestar_attention_drift.argtypes = [I, I, I, I, I, I, I, P, P, F, P, P, I, P, P, Z, P]
    L.polestar_gather_rows.restype = S
    L.polestar_gather_rows.argtypes = [I, I, I, P, P, P, I, P, P]
    L.polestar_scatter_rows.restype = S
    L.polestar_scatter_rows.argtypes = [I, I, I, P, P, P, I, P, P]
    L.polestar_codec_row_bytes.restype = Z
    L.polestar_codec_row_bytes.argtypes = [I, I]
    L.polestar_cluster_means.restype = S
    L.polestar_cluster_means.argtypes = [I, I, I, P, P, I, P, I, P, P]
    L.polestar_codec_encode.restype = S
    L.polestar_codec_encode.argtypes = [I, I, I, I, P, P, P, I, P, I, P, P, P, P]
    L.polestar_codec_gather.restype = S
    L.polestar_codec_gather.argtypes = [I, I, I, I, I, P, P, P, P, I, P, I, P, F, P, P, P]
    Lg = ctypes.c_long
    L.polestar_embed.restype = S
    L.polestar_embed.argtypes = [I, I, I, I, P, I, I, P, I, P, P, P]
    L.polestar_rmsnorm.restype = S
    L.polestar_rmsnorm.argtypes = [I, I, I, I, P, I, I, F, P, I, I, P]
    L.polestar_linear_workspace_size.restype = Z
    L.polestar_linear_workspace_size.argtypes = [I, I, I, I, I]
    L.polestar_linear.restype = S
    L.polestar_linear.argtypes = [I, I, I, I, I, I, I, P, P, P, P, Z, P]
    L.polestar_swiglu.restype = S
    L.polestar_swiglu.argtypes = [I, Lg, I, P, P, P]
    L.polestar_residual_rmsnorm.restype = S
    L.polestar_residual_rmsnorm.argtypes = [I, I, I, I, P, P, F, P, I, I, P]
    L.polestar_linear_swiglu.restype = S
    L.polestar_linear_swiglu.argtypes = [I, I, I, I, I, I, I, P, P, P, P, P, Z, P]
    L.polestar_residual_add.restype = S
    L.polestar_residual_add.argtypes = [I, Lg, P, P, P]
    L.polestar_copy_rows.restype = S
    L.polestar_copy_rows.argtypes = [I, I, I, I, P, P, P, P, I, I, I, P]
    _lib = L
    return L


def _check(fn: str, status: int) -> None:
    if status != OK:
        raise PolestarError(fn, status)


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return FP32
    if t.dtype == torch.bfloat16:
        return BF16
    raise TypeError(f"unsupported dtype {t.dtype}")


def _ptr(t: torch.Tensor | None, dtype: torch.dtype | None = None) -> int | None:
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError("tensor must be on the GPU")
    if not t.is_contiguous():
        raise ValueError("tensor must be contiguous")
    if dtype is not None and t.dtype != dtype:
        raise TypeError(f"expected {dtype}, got {t.dtype}")
    return t.data_ptr()


def _stream(stream) -> int:
    s = torch.cuda.current_stream() if stream is None else stream
    return s.cuda_stream


def _workspace(nbytes: int, device, ws: torch.Tensor | None) -> torch.Tensor | None:
    if nbytes == 0:
        return ws
    if ws is not None and ws.numel() * ws.element_size() >= nbytes:
        return ws
    # the library needs no initialised workspace
    return torch.empty(nbytes, dtype=torch.uint8, device=device)


# ---------------------------------------------------------------------------
# entry points
# ---------------------------------------------------------------------------

def drift(h_cur: torch.Tensor, h_prev: torch.Tensor, out: torch.Tensor | None = None,
          stream=None) -> torch.Tensor:
    """KL(softmax(h_cur[b,i]) || softmax(h_prev[b,i])) -> [batch][seq] float32."""
    b, s, d = h_cur.shape
    if h_prev.shape != h_cur.shape or h_prev.dtype != h_cur.dtype:
        raise ValueError("h_cur and h_prev differ in shape or dtype")
    if out is None:
        out = torch.empty((b, s), dtype=torch.float32, device=h_cur.device)
    _check("polestar_drift", lib().polestar_drift(_dtype_code(h_cur), b, s, d, _ptr(h_cur), _ptr(h_prev),
                                                 _ptr(out, torch.float32), _stream(stream)))
    return out


def select(drift_vals: torch.Tensor, k: int, block_start: int, block_len: int,
           eligible: torch.Tensor | None = None, stale_idx: torch.Tensor | None = None,
           stale_count: torch.Tensor | None = None, stream=None):
    """TopK of the drift over cached positions -> (stale_idx [batch][k] int32, stale_count [batch])."""
    b, s = drift_vals.shape
    dev = drift_vals.device
    if stale_idx is None:
        stale_idx = torch.empty((b, max(k, 0)), dtype=torch.int32, device=dev)
    if stale_count is None:
        stale_count = torch.empty((b,), dtype=torch.int32, device=dev)
    _check("polestar_select", lib().polestar_select(
        b, s, _ptr(drift_vals, torch.float32), _ptr(eligible, torch.uint8), block_start, block_len, k,
        _ptr(stale_idx, torch.int32) if k > 0 else None, _ptr(stale_count, torch.int32), _stream(stream)))
    return stale_idx, stale_count


def refresh_kv_workspace_size(dtype: int, batch: int, d: int, n_kv_heads: int, head_dim: int,
                              k_max: int, block_len: int) -> int:
    return lib().polestar_refresh_kv_workspace_size(dtype, batch, d, n_kv_heads, head_dim, k_max, block_len)


def refresh_kv(h_cur: torch.Tensor, stale_idx: torch.Tensor | None, stale_count: torch.Tensor | None,
               block_start: int, block_len: int, w_k: torch.Tensor, w_v: torch.Tensor,
               k_cache: torch.Tensor, v_cache: torch.Tensor, workspace: torch.Tensor | None = None,
               stream=None) -> None:
    """Re-project rows stale U J_b into k_cache / v_cache in place."""
    b, s, d = h_cur.shape
    _, _, kvh, hd = k_cache.shape
    dt = _dtype_code(h_cur)
    k_max = 0 if stale_idx is None else stale_idx.shape[1]
    ws = _workspace(refresh_kv_workspace_size(dt, b, d, kvh, hd, k_max, block_len), h_cur.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_refresh_kv", lib().polestar_refresh_kv(
        dt, b, s, d, kvh, hd, _ptr(h_cur),
        _ptr(stale_idx, torch.int32) if k_max > 0 else None,
        _ptr(stale_count, torch.int32) if k_max > 0 else None, k_max, block_start, block_len,
        _ptr(w_k, h_cur.dtype), _ptr(w_v, h_cur.dtype), _ptr(k_cache, h_cur.dtype),
        _ptr(v_cache, h_cur.dtype), _ptr(ws), nbytes, _stream(stream)))


def refresh_kv_noalloc(h_cur: torch.Tensor, stale_idx: torch.Tensor | None, stale_count: torch.Tensor | None,
                       block_start: int, block_len: int, w_k: torch.Tensor, w_v: torch.Tensor,
                       k_cache: torch.Tensor, v_cache: torch.Tensor, stream=None) -> None:
    """refresh_kv with the library's own per-GPU scratch array instead of a
    workspace (nothing is allocated; calls overlapping on one GPU race)."""
    b, s, d = h_cur.shape
    _, _, kvh, hd = k_cache.shape
    dt = _dtype_code(h_cur)
    k_max = 0 if stale_idx is None else stale_idx.shape[1]
    _check("polestar_refresh_kv_noalloc", lib().polestar_refresh_kv_noalloc(
        dt, b, s, d, kvh, hd, _ptr(h_cur),
        _ptr(stale_idx, torch.int32) if k_max > 0 else None,
        _ptr(stale_count, torch.int32) if k_max > 0 else None, k_max, block_start, block_len,
        _ptr(w_k, h_cur.dtype), _ptr(w_v, h_cur.dtype), _ptr(k_cache, h_cur.dtype),
        _ptr(v_cache, h_cur.dtype), _stream(stream)))


def refresh_kv_noalloc_max_bytes() -> int:
    return lib().polestar_refresh_kv_noalloc_max_bytes()


def project_qkv_workspace_size(dtype: int, batch: int, d: int, n_heads: int, n_kv_heads: int, head_dim: int,
                               n_rows: int) -> int:
    return lib().polestar_project_qkv_workspace_size(dtype, batch, d, n_heads, n_kv_heads, head_dim, n_rows)


def project_qkv(h_cur: torch.Tensor, row_start: int, n_rows: int, w_q: torch.Tensor, w_k: torch.Tensor,
                w_v: torch.Tensor, q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor,
                workspace: torch.Tensor | None = None, stream=None) -> None:
    """refresh_kv and project_q of the rows [row_start, row_start + n_rows) as one product."""
    b, s, d = h_cur.shape
    _, _, kvh, hd = k_cache.shape
    heads = q.shape[2]
    if tuple(q.shape) != (b, n_rows, heads, hd) or tuple(w_q.shape) != (heads * hd, d):
        raise ValueError("project_qkv: shapes do not match")
    dt = _dtype_code(h_cur)
    ws = _workspace(project_qkv_workspace_size(dt, b, d, heads, kvh, hd, n_rows), h_cur.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_project_qkv", lib().polestar_project_qkv(
        dt, b, s, d, heads, kvh, hd, _ptr(h_cur), row_start, n_rows, _ptr(w_q, h_cur.dtype), _ptr(w_k, h_cur.dtype),
        _ptr(w_v, h_cur.dtype), _ptr(q, h_cur.dtype), _ptr(k_cache, h_cur.dtype), _ptr(v_cache, h_cur.dtype),
        _ptr(ws), nbytes, _stream(stream)))


def project_q_workspace_size(dtype: int, batch: int, d: int, n_heads: int, head_dim: int,
                             block_len: int) -> int:
    return lib().polestar_project_q_workspace_size(dtype, batch, d, n_heads, head_dim, block_len)


def project_q(h_cur: torch.Tensor, w_q: torch.Tensor, block_start: int, block_len: int, n_heads: int,
              out: torch.Tensor | None = None, workspace: torch.Tensor | None = None,
              stream=None) -> torch.Tensor:
    """Q = W_q h_cur[:, J_b] -> [batch][block_len][n_heads][head_dim]."""
    b, s, d = h_cur.shape
    hd = w_q.shape[0] // n_heads
    dt = _dtype_code(h_cur)
    if out is None:
        out = torch.empty((b, block_len, n_heads, hd), dtype=h_cur.dtype, device=h_cur.device)
    ws = _workspace(project_q_workspace_size(dt, b, d, n_heads, hd, block_len), h_cur.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_project_q", lib().polestar_project_q(
        dt, b, s, d, n_heads, hd, block_start, block_len, _ptr(h_cur), _ptr(w_q, h_cur.dtype),
        _ptr(out, h_cur.dtype), _ptr(ws), nbytes, _stream(stream)))
    return out


def attend_workspace_size(dtype: int, batch: int, seq: int, d: int, n_heads: int, n_kv_heads: int,
                          head_dim: int, block_len: int) -> int:
    return lib().polestar_attend_workspace_size(dtype, batch, seq, d, n_heads, n_kv_heads, head_dim, block_len)


def attend(h_cur: torch.Tensor | None, w_q: torch.Tensor | None, k_cache: torch.Tensor,
           v_cache: torch.Tensor, block_start: int, block_len: int, n_heads: int,
           q_buf: torch.Tensor | None = None, out: torch.Tensor | None = None,
           lse: torch.Tensor | None = None, scale: float = 0.0,
           workspace: torch.Tensor | None = None, stream=None):
    """Bidirectional attention of the active block over the whole cache.

    With w_q, Q = W_q h_cur[:, J_b] is projected into q_buf first; without,
    q_buf must hold Q.  Returns (out, q_buf)."""
    b, s, kvh, hd = k_cache.shape
    dt = _dtype_code(k_cache)
    dev = k_cache.device
    d = h_cur.shape[2] if h_cur is not None else n_heads * hd
    if q_buf is None:
        q_buf = torch.empty((b, block_len, n_heads, hd), dtype=k_cache.dtype, device=dev)
    if out is None:
        out = torch.empty((b, block_len, n_heads, hd), dtype=k_cache.dtype, device=dev)
    ws = _workspace(attend_workspace_size(dt, b, s, d, n_heads, kvh, hd, block_len), dev, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_attend", lib().polestar_attend(
        dt, b, s, d, n_heads, kvh, hd, block_start, block_len,
        _ptr(h_cur) if w_q is not None else None, _ptr(w_q), _ptr(q_buf, k_cache.dtype),
        _ptr(k_cache), _ptr(v_cache, k_cache.dtype), float(scale), _ptr(out, k_cache.dtype),
        _ptr(lse, torch.float32), _ptr(ws), nbytes, _stream(stream)))
    return out, q_buf


def commit_workspace_size(dtype: int, batch: int, block_len: int, vocab: int) -> int:
    return lib().polestar_commit_workspace_size(dtype, batch, block_len, vocab)


def commit(logits: torch.Tensor, masked: torch.Tensor, drift_vals: torch.Tensor | None,
           block_start: int, hist: torch.Tensor | None, hist_len: torch.Tensor | None,
           mask_token_id: int = -1, tau_s: float = DEFAULT_TAU_S, alpha: float = DEFAULT_ALPHA,
           force_one: bool = False, token: torch.Tensor | None = None,
           conf: torch.Tensor | None = None, commit_out: torch.Tensor | None = None,
           workspace: torch.Tensor | None = None, stream=None):
    """Polestar-Commit of the current block -> (token int32, conf float32, commit uint8)."""
    b, nq, vocab = logits.shape
    dt = _dtype_code(logits)
    dev = logits.device
    seq = drift_vals.shape[1] if drift_vals is not None else 0
    h = hist.shape[1] if hist is not None else 0
    if token is None:
        token = torch.empty((b, nq), dtype=torch.int32, device=dev)
    if conf is None:
        conf = torch.empty((b, nq), dtype=torch.float32, device=dev)
    if commit_out is None:
        commit_out = torch.empty((b, nq), dtype=torch.uint8, device=dev)
    ws = _workspace(commit_workspace_size(dt, b, nq, vocab), dev, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_commit", lib().polestar_commit(
        dt, b, nq, vocab, _ptr(logits), _ptr(masked, torch.uint8), _ptr(drift_vals, torch.float32), seq,
        block_start, _ptr(hist, torch.float32), _ptr(hist_len, torch.int32), h, mask_token_id,
        float(tau_s), float(alpha), int(bool(force_one)), _ptr(token, torch.int32),
        _ptr(conf, torch.float32), _ptr(commit_out, torch.uint8), _ptr(ws), nbytes, _stream(stream)))
    return token, conf, commit_out


def suffix_commit(logits: torch.Tensor, masked: torch.Tensor, eligible: torch.Tensor,
                  mask_token_id: int = -1, tau_s: float = DEFAULT_TAU_S, token: torch.Tensor | None = None,
                  conf: torch.Tensor | None = None, commit_out: torch.Tensor | None = None,
                  workspace: torch.Tensor | None = None, stream=None):
    """Suffix-block commit of the packet rows -> (token int32, conf float32, commit uint8)."""
    b, n, vocab = logits.shape
    dt = _dtype_code(logits)
    dev = logits.device
    if token is None:
        token = torch.empty((b, n), dtype=torch.int32, device=dev)
    if conf is None:
        conf = torch.empty((b, n), dtype=torch.float32, device=dev)
    if commit_out is None:
        commit_out = torch.empty((b, n), dtype=torch.uint8, device=dev)
    ws = _workspace(commit_workspace_size(dt, b, n, vocab), dev, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_suffix_commit", lib().polestar_suffix_commit(
        dt, b, n, vocab, _ptr(logits), _ptr(masked, torch.uint8), _ptr(eligible, torch.uint8), mask_token_id,
        float(tau_s), _ptr(token, torch.int32), _ptr(conf, torch.float32), _ptr(commit_out, torch.uint8),
        _ptr(ws), nbytes, _stream(stream)))
    return token, conf, commit_out


# ---------------------------------------------------------------------------
# the rest of a layer stack (embedding, RMSNorm, projections, SwiGLU)
# ---------------------------------------------------------------------------

def embed(ids: torch.Tensor, lo: int, n_rows: int, tok_emb: torch.Tensor, pos_emb: torch.Tensor,
          x: torch.Tensor, stream=None) -> torch.Tensor:
    """x[b][r] = tok_emb[ids[b][lo + r]] + pos_emb[lo + r]; x is [batch][n_rows][d] float32."""
    b, seq = ids.shape
    vocab, d = tok_emb.shape
    if tuple(x.shape) != (b, n_rows, d):
        raise ValueError("x must be [batch][n_rows][d]")
    _check("polestar_embed", lib().polestar_embed(
        _dtype_code(tok_emb), b, seq, d, _ptr(ids, torch.int32), lo, n_rows, _ptr(tok_emb), vocab,
        _ptr(pos_emb, tok_emb.dtype), _ptr(x, torch.float32), _stream(stream)))
    return x


def rmsnorm(x: torch.Tensor, x_start: int, n_rows: int, out: torch.Tensor, out_start: int,
            eps: float = 1e-5, stream=None) -> torch.Tensor:
    """out[b][out_start + r] = RMSNorm(x[b][x_start + r]) (unit gain), rounded to out's dtype."""
    b, x_seq, d = x.shape
    if out.shape[0] != b or out.shape[2] != d:
        raise ValueError("x and out differ in batch or width")
    _check("polestar_rmsnorm", lib().polestar_rmsnorm(
        _dtype_code(out), b, n_rows, d, _ptr(x, torch.float32), x_seq, x_start, float(eps), _ptr(out),
        out.shape[1], out_start, _stream(stream)))
    return out


def linear_workspace_size(dtype: int, batch: int, n_rows: int, n_out: int, n_in: int) -> int:
    return lib().polestar_linear_workspace_size(dtype, batch, n_rows, n_out, n_in)


def linear(x: torch.Tensor, row_start: int, n_rows: int, w: torch.Tensor, y: torch.Tensor,
           workspace: torch.Tensor | None = None, stream=None) -> torch.Tensor:
    """y[b][r] = W x[b][row_start + r]; x [batch][seq][n_in], w [n_out][n_in], y [batch][n_rows][n_out]."""
    b, seq, n_in = x.shape
    n_out = w.shape[0]
    if tuple(y.shape) != (b, n_rows, n_out) or w.shape[1] != n_in:
        raise ValueError("linear: shapes do not match")
    dt = _dtype_code(x)
    ws = _workspace(linear_workspace_size(dt, b, n_rows, n_out, n_in), x.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_linear", lib().polestar_linear(
        dt, b, seq, n_in, n_out, row_start, n_rows, _ptr(x), _ptr(w, x.dtype), _ptr(y, x.dtype), _ptr(ws), nbytes,
        _stream(stream)))
    return y


def swiglu(gate_up: torch.Tensor, out: torch.Tensor, stream=None) -> torch.Tensor:
    """out[..., f] = silu(gate_up[..., f]) * gate_up[..., F + f], F = out.shape[-1]."""
    f = out.shape[-1]
    rows = out.numel() // f
    if gate_up.numel() != 2 * out.numel():
        raise ValueError("gate_up must hold 2*F values per row")
    _check("polestar_swiglu", lib().polestar_swiglu(_dtype_code(out), rows, f, _ptr(gate_up, out.dtype),
                                                   _ptr(out), _stream(stream)))
    return out


def residual_add(x: torch.Tensor, y: torch.Tensor, stream=None) -> torch.Tensor:
    """x += y (float32 += dtype), same number of elements."""
    if x.numel() != y.numel():
        raise ValueError("residual_add: sizes differ")
    _check("polestar_residual_add", lib().polestar_residual_add(
        _dtype_code(y), x.numel(), _ptr(x, torch.float32), _ptr(y), _stream(stream)))
    return x


def residual_rmsnorm(x: torch.Tensor, y: torch.Tensor, out: torch.Tensor, out_start: int, eps: float = 1e-5,
                     stream=None) -> torch.Tensor:
    """x += y, then out[b][out_start + r] = RMSNorm(x[b][r]); x, y [batch][n_rows][d], out [batch][seq][d]."""
    b, n, d = x.shape
    if tuple(y.shape) != (b, n, d) or out.shape[0] != b or out.shape[2] != d:
        raise ValueError("residual_rmsnorm: shapes do not match")
    _check("polestar_residual_rmsnorm", lib().polestar_residual_rmsnorm(
        _dtype_code(out), b, n, d, _ptr(x, torch.float32), _ptr(y, out.dtype), eps, _ptr(out), out.shape[1], out_start,
        _stream(stream)))
    return out


def linear_swiglu(x: torch.Tensor, row_start: int, n_rows: int, w_gate_up: torch.Tensor, gate_up: torch.Tensor,
                  out: torch.Tensor, workspace: torch.Tensor | None = None, stream=None) -> torch.Tensor:
    """out[b][r] = silu(gate) * up of W_gate_up x[b][row_start + r]; gate_up [batch][n_rows][2F] is scratch."""
    b, seq, n_in = x.shape
    f = out.shape[-1]
    if (tuple(out.shape) != (b, n_rows, f) or gate_up.numel() != 2 * out.numel()
            or tuple(w_gate_up.shape) != (2 * f, n_in)):
        raise ValueError("linear_swiglu: shapes do not match")
    dt = _dtype_code(x)
    ws = _workspace(linear_workspace_size(dt, b, n_rows, 2 * f, n_in), x.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_linear_swiglu", lib().polestar_linear_swiglu(
        dt, b, seq, n_in, f, row_start, n_rows, _ptr(x), _ptr(w_gate_up, x.dtype), _ptr(gate_up, x.dtype),
        _ptr(out, x.dtype), _ptr(ws), nbytes, _stream(stream)))
    return out


def copy_rows(src: torch.Tensor, dst: torch.Tensor, stale_idx: torch.Tensor | None,
              stale_count: torch.Tensor | None, block_start: int, block_len: int, stream=None) -> None:
    """dst rows = src rows for the stale set and the block (the rows refresh_kv rewrites)."""
    b, seq, d = src.shape
    k_max = 0 if stale_idx is None else stale_idx.shape[1]
    _check("polestar_copy_rows", lib().polestar_copy_rows(
        _dtype_code(src), b, seq, d, _ptr(src), _ptr(dst, src.dtype),
        _ptr(stale_idx, torch.int32) if k_max > 0 else None,
        _ptr(stale_count, torch.int32) if k_max > 0 else None, k_max, block_start, block_len, _stream(stream)))


def gather_rows(src: torch.Tensor, idx: torch.Tensor, count: torch.Tensor, dst: torch.Tensor, stream=None):
    """dst[b][r] = src[b][idx[b][r]] for r < count[b], zero rows after;
    src [batch][seq][...], dst [batch][k_max][...] of the same row shape and dtype."""
    b, seq = src.shape[0], src.shape[1]
    k_max = idx.shape[1]
    rb = src[0, 0].numel() * src.element_size()
    if dst.shape[0] != b or dst.shape[1] != k_max or dst[0, 0].numel() * dst.element_size() != rb:
        raise ValueError("gather_rows: shapes do not match")
    _check("polestar_gather_rows", lib().polestar_gather_rows(
        b, seq, rb, _ptr(src), _ptr(idx, torch.int32), _ptr(count, torch.int32), k_max, _ptr(dst, src.dtype),
        _stream(stream)))
    return dst


def scatter_rows(src: torch.Tensor, idx: torch.Tensor, count: torch.Tensor, dst: torch.Tensor, stream=None):
    """dst[b][idx[b][r]] = src[b][r] for r < count[b]; src [batch][k_max][...], dst [batch][seq][...]."""
    b, seq = dst.shape[0], dst.shape[1]
    k_max = idx.shape[1]
    rb = dst[0, 0].numel() * dst.element_size()
    if src.shape[0] != b or src.shape[1] != k_max or src[0, 0].numel() * src.element_size() != rb:
        raise ValueError("scatter_rows: shapes do not match")
    _check("polestar_scatter_rows", lib().polestar_scatter_rows(
        b, seq, rb, _ptr(src, dst.dtype), _ptr(idx, torch.int32), _ptr(count, torch.int32), k_max, _ptr(dst),
        _stream(stream)))
    return dst


def codec_row_bytes(fmt: int, d: int) -> int:
    return lib().polestar_codec_row_bytes(fmt, d)


def cluster_means(x: torch.Tensor, win_idx: torch.Tensor, labels: torch.Tensor, n_clusters: int,
                  means: torch.Tensor | None = None, stream=None) -> torch.Tensor:
    """Per cluster the mean of its window members' rows of x [b][seq][d] (float32) -> [b][K][d]."""
    b, seq, d = x.shape
    if means is None:
        means = torch.empty((b, n_clusters, d), dtype=torch.float32, device=x.device)
    _check("polestar_cluster_means", lib().polestar_cluster_means(
        b, seq, d, _ptr(x, torch.float32), _ptr(win_idx, torch.int32), win_idx.shape[1], _ptr(labels, torch.int32),
        n_clusters, _ptr(means, torch.float32), _stream(stream)))
    return means


def codec_encode(fmt: int, x: torch.Tensor, idx: torch.Tensor, count: torch.Tensor, labels: torch.Tensor,
                 means: torch.Tensor, codes: torch.Tensor, scales: torch.Tensor, stream=None) -> None:
    """Codes and scales of the rows idx (residuals of x to their cluster mean), by position."""
    b, seq, d = x.shape
    _check("polestar_codec_encode", lib().polestar_codec_encode(
        fmt, b, seq, d, _ptr(x, torch.float32), _ptr(idx, torch.int32), _ptr(count, torch.int32), idx.shape[1],
        _ptr(labels, torch.int32), means.shape[1], _ptr(means, torch.float32), _ptr(codes, torch.uint8),
        _ptr(scales, torch.uint8), _stream(stream)))


def codec_gather(fmt: int, codes: torch.Tensor, scales: torch.Tensor, idx: torch.Tensor, count: torch.Tensor,
                 labels: torch.Tensor, means: torch.Tensor, x_out: torch.Tensor, h_out: torch.Tensor | None = None,
                 eps: float = 1e-5, stream=None) -> None:
    """x_out[b][r] = mean + decoded residual of row idx[b][r]; h_out = its RMSNorm (fused)."""
    b, seq = labels.shape
    k_max = idx.shape[1]
    d = x_out.shape[2]
    dt = _dtype_code(h_out) if h_out is not None else BF16
    _check("polestar_codec_gather", lib().polestar_codec_gather(
        fmt, dt, b, seq, d, _ptr(codes, torch.uint8), _ptr(scales, torch.uint8), _ptr(idx, torch.int32),
        _ptr(count, torch.int32), k_max, _ptr(labels, torch.int32), means.shape[1], _ptr(means, torch.float32),
        float(eps), _ptr(x_out, torch.float32), _ptr(h_out), _stream(stream)))


# ---------------------------------------------------------------------------
# one layer step with preallocated buffers
# ---------------------------------------------------------------------------

# ---------------------------------------------------------------------------
# clustered proxy drift
# ---------------------------------------------------------------------------

def window_positions(seq: int, block_start: int, block_len: int, prefix: int, suffix: int) -> list:
    """The local window around the active block: [start - prefix, start) and
    [end, end + suffix), clipped to the sequence."""
    lo, hi = max(0, block_start - prefix), min(seq, block_start + block_len + suffix)
    return list(range(lo, block_start)) + list(range(block_start + block_len, hi))


def cluster(h: torch.Tensor, win_idx: torch.Tensor, n_clusters: int, iters: int = 10, stream=None):
    """Spherical K-means of the window's hidden states -> (labels [b][seq],
    sums [b][K][d], counts [b][K], centroids [b][K][d])."""
    b, seq, d = h.shape
    dev = h.device
    n_win = win_idx.shape[1]
    labels = torch.empty((b, seq), dtype=torch.int32, device=dev)
    sums = torch.empty((b, n_clusters, d), dtype=torch.float32, device=dev)
    counts = torch.empty((b, n_clusters), dtype=torch.int32, device=dev)
    cents = torch.empty((b, n_clusters, d), dtype=torch.float32, device=dev)
    _check("polestar_cluster", lib().polestar_cluster(
        _dtype_code(h), b, seq, d, _ptr(h), _ptr(win_idx, torch.int32), n_win, n_clusters, iters,
        _ptr(labels), _ptr(sums), _ptr(counts), _ptr(cents), _stream(stream)))
    return labels, sums, counts, cents


def proxy_drift_workspace_size(dtype: int, batch: int, seq: int, d: int, n_heads: int, head_dim: int,
                               n_clusters: int) -> int:
    return lib().polestar_proxy_drift_workspace_size(dtype, batch, seq, d, n_heads, head_dim, n_clusters)


def proxy_drift(sums: torch.Tensor, counts: torch.Tensor, w_q: torch.Tensor, k_cache: torch.Tensor,
                n_heads: int, scores: torch.Tensor, lse: torch.Tensor, first: bool,
                drift_out: torch.Tensor | None = None, scale: float = 0.0,
                workspace: torch.Tensor | None = None, stream=None) -> torch.Tensor:
    """Drift per cluster [b][K]; scores [b][K][H][seq] and lse [b][K][H] are
    the previous step's on entry and this step's on return."""
    b, K, d = sums.shape
    _, seq, kvh, hd = k_cache.shape
    dt = _dtype_code(k_cache)
    if drift_out is None:
        drift_out = torch.empty((b, K), dtype=torch.float32, device=sums.device)
    ws = _workspace(proxy_drift_workspace_size(dt, b, seq, d, n_heads, hd, K), sums.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_proxy_drift", lib().polestar_proxy_drift(
        dt, b, seq, d, n_heads, kvh, hd, K, _ptr(sums, torch.float32), _ptr(counts, torch.int32),
        _ptr(w_q, k_cache.dtype), _ptr(k_cache), float(scale), _ptr(scores, torch.float32),
        _ptr(lse, torch.float32), int(bool(first)), _ptr(drift_out, torch.float32), _ptr(ws), nbytes,
        _stream(stream)))
    return drift_out


def attention_drift_workspace_size(batch: int, seq: int, n_rows: int, n_heads: int) -> int:
    return lib().polestar_attention_drift_workspace_size(batch, seq, n_rows, n_heads)


def attention_drift(q: torch.Tensor, k_cache: torch.Tensor, scores: torch.Tensor, lse: torch.Tensor, first: bool,
                    drift_out: torch.Tensor | None = None, scale: float = 0.0,
                    workspace: torch.Tensor | None = None, stream=None) -> torch.Tensor:
    """KL of each query row's attention distribution against the previous
    step's, averaged over heads -> [batch][n_rows]; scores [b][R][H][seq] and
    lse [b][R][H] are the previous step's on entry and this step's on return."""
    b, R, H, hd = q.shape
    _, seq, kvh, _ = k_cache.shape
    if drift_out is None:
        drift_out = torch.empty((b, R), dtype=torch.float32, device=q.device)
    ws = _workspace(attention_drift_workspace_size(b, seq, R, H), q.device, workspace)
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    _check("polestar_attention_drift", lib().polestar_attention_drift(
        _dtype_code(q), b, seq, R, H, kvh, hd, _ptr(q), _ptr(k_cache, q.dtype), float(scale),
        _ptr(scores, torch.float32), _ptr(lse, torch.float32), int(bool(first)), _ptr(drift_out, torch.float32),
        _ptr(ws), nbytes, _stream(stream)))
    return drift_out


def cluster_select(labels: torch.Tensor, drift_vals: torch.Tensor, k_top: int, k_max: int,
                   stale_idx: torch.Tensor | None = None, stale_count: torch.Tensor | None = None,
                   stream=None):
    """Members of the k_top clusters of largest drift -> (stale_idx [b][k_max], stale_count [b])."""
    b, seq = labels.shape
    K = drift_vals.shape[1]
    dev = labels.device
    if stale_idx is None:
        stale_idx = torch.empty((b, k_max), dtype=torch.int32, device=dev)
    if stale_count is None:
        stale_count = torch.empty((b,), dtype=torch.int32, device=dev)
    _check("polestar_cluster_select", lib().polestar_cluster_select(
        b, seq, _ptr(labels, torch.int32), K, _ptr(drift_vals, torch.float32), k_top,
        _ptr(stale_idx, torch.int32) if k_max > 0 else None, k_max, _ptr(stale_count, torch.int32),
        _stream(stream)))
    return stale_idx, stale_count


def cluster_update(h_new: torch.Tensor, h_old: torch.Tensor, labels: torch.Tensor,
                   stale_idx: torch.Tensor, stale_count: torch.Tensor, sums: torch.Tensor,
                   stream=None) -> None:
    """sums[label(p)] += h_new[p] - h_old[p] for the refreshed window rows."""
    b, seq, d = h_new.shape
    K = sums.shape[1]
    k_max = stale_idx.shape[1]
    _check("polestar_cluster_update", lib().polestar_cluster_update(
        _dtype_code(h_new), b, seq, d, _ptr(h_new), _ptr(h_old, h_new.dtype), _ptr(labels, torch.int32), K,
        _ptr(stale_idx, torch.int32) if k_max > 0 else None, _ptr(stale_count, torch.int32), k_max,
        _ptr(sums, torch.float32), _stream(stream)))


def _event_handle(ev) -> int | None:
    """Raw hipEvent_t of a torch.cuda.Event (created by recording it once), or
    an int that already is one (an event created through the HIP runtime)."""
    if ev is None:
        return None
    if isinstance(ev, int):
        return ev
    if not ev.cuda_event:
        ev.record()
    return ev.cuda_event


def step_args(*, h_cur, h_prev, w_q, w_k, w_v, k_cache, v_cache, logits, masked, hist, hist_len,
              drift_out, stale_idx, stale_count, q, out, lse, token, conf, commit_out, k: int,
              block_start: int, block_len: int, n_heads: int, eligible=None, mask_token_id: int = -1,
              tau_s: float = DEFAULT_TAU_S, alpha: float = DEFAULT_ALPHA, force_one: bool = False,
              scale: float = 0.0) -> StepArgs:
    """polestar_step_args for one layer step (checks dtypes and devices)."""
    b, seq, d = h_cur.shape
    _, _, kvh, hd = k_cache.shape
    dt = h_cur.dtype
    a = StepArgs()
    a.dtype = _dtype_code(h_cur)
    a.batch, a.seq, a.d = b, seq, d
    a.n_heads, a.n_kv_heads, a.head_dim = n_heads, kvh, hd
    a.block_start, a.block_len = block_start, block_len
    a.vocab = logits.shape[2]
    a.k = k
    a.h = hist.shape[1] if hist is not None else 0
    a.mask_token_id = mask_token_id
    a.force_one = int(bool(force_one))
    a.tau_s, a.alpha, a.scale = float(tau_s), float(alpha), float(scale)
    a.h_cur, a.h_prev = _ptr(h_cur), _ptr(h_prev, dt)
    a.eligible = _ptr(eligible, torch.uint8)
    a.w_q, a.w_k, a.w_v = _ptr(w_q, dt), _ptr(w_k, dt), _ptr(w_v, dt)
    a.k_cache, a.v_cache = _ptr(k_cache, dt), _ptr(v_cache, dt)
    a.logits, a.masked = _ptr(logits, dt), _ptr(masked, torch.uint8)
    a.hist, a.hist_len = _ptr(hist, torch.float32), _ptr(hist_len, torch.int32)
    a.drift = _ptr(drift_out, torch.float32)
    a.stale_idx = _ptr(stale_idx, torch.int32) if k > 0 else None
    a.stale_count = _ptr(stale_count, torch.int32)
    a.q, a.out = _ptr(q, dt), _ptr(out, dt)
    a.lse = _ptr(lse, torch.float32)
    a.token, a.conf, a.commit = _ptr(token, torch.int32), _ptr(conf, torch.float32), _ptr(commit_out, torch.uint8)
    return a


def step_workspace_size(args: StepArgs) -> int:
    return lib().polestar_step_workspace_size(ctypes.byref(args))


def step(args: StepArgs, workspace: torch.Tensor, refresh_events=None, stream=None) -> None:
    """polestar_step: the whole layer step; refresh_events = (begin, end)
    pair of torch.cuda.Event or raw hipEvent_t recorded around the K/V
    refresh, or None."""
    ev0, ev1 = refresh_events if refresh_events is not None else (None, None)
    nbytes = workspace.numel() * workspace.element_size()
    _check("polestar_step", lib().polestar_step(ctypes.byref(args), _ptr(workspace), nbytes,
                                                _event_handle(ev0), _event_handle(ev1), _stream(stream)))


class Step:
    """One layer step on buffers allocated once, on the current stream:
    drift -> select -> refresh_kv -> project_q -> attend -> commit, through
    polestar_step (run) or as six separate calls (run_calls).

    (The query projection reads only h_cur and W_q and could run on a second
    stream; measured on MI355X, the cross-stream event waits cost more than
    the overlap saves at these sizes, so the step stays on one stream.)
    """

    def __init__(self, *, batch: int, seq: int, d: int, n_heads: int, n_kv_heads: int,
                 head_dim: int, block_start: int, block_len: int, vocab: int, k: int,
                 dtype: torch.dtype, hist_depth: int = DEFAULT_HISTORY, device="cuda"):
        self.shape = dict(batch=batch, seq=seq, d=d, n_heads=n_heads, n_kv_heads=n_kv_heads,
                          head_dim=head_dim, block_start=block_start, block_len=block_len,
                          vocab=vocab, k=k)
        dt = FP32 if dtype == torch.float32 else BF16
        dev = torch.device(device)
        f = dict(device=dev)
        self.drift = torch.empty((batch, seq), dtype=torch.float32, **f)
        self.stale_idx = torch.empty((batch, k), dtype=torch.int32, **f) if k > 0 else None
        self.stale_count = torch.empty((batch,), dtype=torch.int32, **f)
        self.q_buf = torch.empty((batch, block_len, n_heads, head_dim), dtype=dtype, **f)
        self.out = torch.empty((batch, block_len, n_heads, head_dim), dtype=dtype, **f)
        self.lse = torch.empty((batch, n_heads, block_len), dtype=torch.float32, **f)
        self.token = torch.empty((batch, block_len), dtype=torch.int32, **f)
        self.conf = torch.empty((batch, block_len), dtype=torch.float32, **f)
        self.commit = torch.empty((batch, block_len), dtype=torch.uint8, **f)
        self.ws_refresh = _workspace(refresh_kv_workspace_size(dt, batch, d, n_kv_heads, head_dim, k, block_len), dev, None)
        self.ws_q = _workspace(project_q_workspace_size(dt, batch, d, n_heads, head_dim, block_len), dev, None)
        self.ws_attend = _workspace(attend_workspace_size(dt, batch, seq, d, n_heads, n_kv_heads, head_dim, block_len), dev, None)
        self.ws_commit = _workspace(commit_workspace_size(dt, batch, block_len, vocab), dev, None)
        self.ws_step = None

    def prepare(self, h_cur, h_prev, w_q, w_k, w_v, k_cache, v_cache, logits, masked, hist, hist_len,
                *, mask_token_id=-1, tau_s=DEFAULT_TAU_S, alpha=DEFAULT_ALPHA, force_one=False,
                eligible=None) -> StepArgs:
        """polestar_step_args for these inputs and this step's outputs (build
        once, launch many times while the tensors stay the same)."""
        s = self.shape
        args = step_args(h_cur=h_cur, h_prev=h_prev, w_q=w_q, w_k=w_k, w_v=w_v, k_cache=k_cache,
                         v_cache=v_cache, logits=logits, masked=masked, hist=hist, hist_len=hist_len,
                         drift_out=self.drift, stale_idx=self.stale_idx, stale_count=self.stale_count,
                         q=self.q_buf, out=self.out, lse=self.lse, token=self.token, conf=self.conf,
                         commit_out=self.commit, k=s["k"], block_start=s["block_start"],
                         block_len=s["block_len"], n_heads=s["n_heads"], eligible=eligible,
                         mask_token_id=mask_token_id, tau_s=tau_s, alpha=alpha, force_one=force_one)
        need = step_workspace_size(args)
        if self.ws_step is None or self.ws_step.numel() < need:
            self.ws_step = _workspace(need, self.drift.device, None)
        return args

    def launch(self, args: StepArgs, refresh_events=None):
        """polestar_step on prepared arguments."""
        step(args, self.ws_step, refresh_events)
        return self

    def run(self, h_cur, h_prev, w_q, w_k, w_v, k_cache, v_cache, logits, masked, hist, hist_len,
            *, mask_token_id=-1, tau_s=DEFAULT_TAU_S, alpha=DEFAULT_ALPHA, force_one=False,
            eligible=None, refresh_events=None):
        """The step through polestar_step (fused launches)."""
        args = self.prepare(h_cur, h_prev, w_q, w_k, w_v, k_cache, v_cache, logits, masked, hist, hist_len,
                            mask_token_id=mask_token_id, tau_s=tau_s, alpha=alpha, force_one=force_one,
                            eligible=eligible)
        return self.launch(args, refresh_events)

    def run_calls(self, h_cur, h_prev, w_q, w_k, w_v, k_cache, v_cache, logits, masked, hist, hist_len,
                  *, mask_token_id=-1, tau_s=DEFAULT_TAU_S, alpha=DEFAULT_ALPHA, force_one=False,
                  eligible=None):
        """The same step as six separate calls."""
        s = self.shape
        drift(h_cur, h_prev, out=self.drift)
        select(self.drift, s["k"], s["block_start"], s["block_len"], eligible, self.stale_idx,
               self.stale_count)
        refresh_kv(h_cur, self.stale_idx, self.stale_count, s["block_start"], s["block_len"],
                   w_k, w_v, k_cache, v_cache, workspace=self.ws_refresh)
        project_q(h_cur, w_q, s["block_start"], s["block_len"], s["n_heads"], out=self.q_buf,
                  workspace=self.ws_q)
        attend(None, None, k_cache, v_cache, s["block_start"], s["block_len"], s["n_heads"],
               q_buf=self.q_buf, out=self.out, lse=self.lse, workspace=self.ws_attend)
        commit(logits, masked, self.drift, s["block_start"], hist, hist_len, mask_token_id,
               tau_s, alpha, force_one, self.token, self.conf, self.commit, workspace=self.ws_commit)
        return self
