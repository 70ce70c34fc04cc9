"""Thin binding of the C-ABI library declared in include/lx.h.

Only argument marshalling happens here: torch tensors supply device pointers
and the current HIP stream; every step of the operators runs inside the
library's kernels.  The calls of a training step marshal in native code
(csrc/lx_call.cpp), the others through ctypes.  Importing this module fails
loudly when the library has not been built (run
`python paper_2510_15964_amd/build.py`); there is no CPU or PyTorch fallback.
"""
from __future__ import annotations

import ctypes as C
import importlib.machinery
import importlib.util
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "liblx_sparse.so")

CALL_PATH = os.path.join(_HERE, "_lx_call" + importlib.machinery.EXTENSION_SUFFIXES[0])      # built for this interpreter

for _path in (LIB_PATH, CALL_PATH):
    if not os.path.exists(_path):
        raise ImportError(
            f"{_path} is missing: build the HIP library first "
            "(python paper_2510_15964_amd/build.py). There is no fallback path.")

_lib = C.CDLL(LIB_PATH)

LX_OK, LX_ERR_INVALID_ARG, LX_ERR_UNSUPPORTED, LX_ERR_WORKSPACE, LX_ERR_RUNTIME = range(5)
LX_F32, LX_BF16, LX_F16 = 0, 1, 2

EXPORTS = (
    "lx_status_string", "lx_mask_compact", "lx_mask_compact_pair", "lx_mask_compact_batch", "lx_ffn_pack_weights",
    "lx_ffn_gather_weight_blocks",
    "lx_sparse_ffn_fwd_workspace_bytes", "lx_sparse_ffn_bwd_workspace_bytes",
    "lx_sparse_ffn_split_workspace_bytes",
    "lx_sparse_ffn_fwd", "lx_sparse_ffn_bwd_dx", "lx_sparse_attn_bwd_workspace_bytes",
    "lx_sparse_attn_fwd", "lx_sparse_attn_bwd_dx", "lx_sparse_attn_bwd_dx_noalloc", "lx_profile_begin", "lx_profile_end",
    "lx_attn_set_rows_per_workgroup", "lx_ffn_set_token_tiles_per_workgroup", "lx_mlp_predict_mask", "lx_attn_combine_patterns",
    "lx_sparse_ffn_lora_fwd_workspace_bytes", "lx_sparse_ffn_lora_bwd_workspace_bytes",
    "lx_sparse_ffn_lora_fwd", "lx_sparse_ffn_lora_bwd", "lx_probe_mfma_rate", "lx_probe_stream_copy",
)
(LX_K_COMPACT, LX_K_FFN_UP, LX_K_FFN_DOWN, LX_K_FFN_DH, LX_K_FFN_DX, LX_K_ATTN_FWD,
 LX_K_ATTN_BWD_DQ, LX_K_ATTN_BWD_DKV, LX_K_TRANSPOSE, LX_K_PREDICT, LX_K_COMBINE,
 LX_K_LORA) = range(12)
KERNEL_NAMES = ("compact", "ffn_up", "ffn_down", "ffn_dh", "ffn_dx", "attn_fwd", "attn_bwd_dq",
                "attn_bwd_dkv", "transpose", "predict", "combine", "lora")


class lx_blocklist(C.Structure):
    _fields_ = [("rows", C.c_int32), ("cols", C.c_int32), ("row_ptr", C.c_void_p),
                ("col_idx", C.c_void_p), ("nnz_cap", C.c_int32)]


_i32, _i64, _vp, _sz, _f = C.c_int32, C.c_int64, C.c_void_p, C.c_size_t, C.c_float


class lx_compact_job(C.Structure):
    _fields_ = [("mask", C.c_void_p), ("batch", C.c_int32), ("rows", C.c_int32),
                ("cols", C.c_int32), ("batch_stride", C.c_int64), ("row_stride", C.c_int64),
                ("col_stride", C.c_int64), ("row_ptr", C.c_void_p), ("col_idx", C.c_void_p),
                ("col_idx_cap", C.c_int32)]
_blp = C.POINTER(lx_blocklist)
_lib.lx_status_string.restype = C.c_char_p
_lib.lx_status_string.argtypes = [C.c_int]
_lib.lx_mask_compact.argtypes = [_vp, _i32, _i32, _i32, _i64, _i64, _i64, _vp, _vp, _i32, _vp]
_lib.lx_mask_compact_pair.argtypes = [_vp, _i32, _i32, _i32, _i64, _i64, _i64, _vp, _vp, _vp, _vp,
                                      _i32, _vp]
_lib.lx_mask_compact_batch.argtypes = [C.POINTER(lx_compact_job), _i32, _vp]
_lib.lx_ffn_pack_weights.argtypes = [C.c_int, _i32, _i32, _vp, _vp, _vp, _vp, _vp]
_lib.lx_ffn_gather_weight_blocks.argtypes = [C.c_int, _i32, _i32, _i32, _vp, _blp, _vp, _vp, _vp, _vp]
for _n in ("lx_sparse_ffn_fwd_workspace_bytes", "lx_sparse_ffn_bwd_workspace_bytes"):
    getattr(_lib, _n).restype = _sz
    getattr(_lib, _n).argtypes = [C.c_int, _i32, _i32, _i32, _i32, _i32, _i32, _i32]
_lib.lx_sparse_ffn_split_workspace_bytes.restype = _sz
_lib.lx_sparse_ffn_split_workspace_bytes.argtypes = [C.c_int, _i32, _i32, _i32, _blp]
_lib.lx_sparse_attn_bwd_workspace_bytes.restype = _sz
_lib.lx_sparse_attn_bwd_workspace_bytes.argtypes = [C.c_int, _i32, _i32, _i32, _i32]
_lib.lx_sparse_ffn_fwd.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _i32, _vp, _vp, _vp, _vp, _vp,
                                   _blp, _vp, _vp, _vp, _sz, _vp]
_lib.lx_sparse_ffn_bwd_dx.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _i32, _vp, _vp, _vp, _vp,
                                      _vp, _vp, _blp, _vp, _vp, _sz, _vp]
_lib.lx_sparse_attn_fwd.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _f, _i32, _vp, _vp, _vp,
                                    C.POINTER(_i64), _blp, _i32, _vp, _vp, _vp, _vp]
_lib.lx_sparse_attn_bwd_dx.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _f, _i32, _vp, _vp, _vp,
                                       _vp, _vp, _vp, C.POINTER(_i64), _blp, _blp, _i32, _vp, _vp,
                                       _vp, _vp, _vp, _sz, _vp]
_lib.lx_sparse_attn_bwd_dx_noalloc.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _f, _i32, _vp, _vp, _vp,
                                               _vp, _vp, _vp, C.POINTER(_i64), _blp, _blp, _i32, _vp,
                                               _vp, _vp, _vp, _vp]

_lib.lx_probe_mfma_rate.argtypes = [_i32, _vp, C.POINTER(C.c_double), _vp]
_lib.lx_probe_stream_copy.argtypes = [_vp, _vp, _sz, _vp]
_lib.lx_profile_begin.argtypes = [_i32, _i32]
_lib.lx_profile_end.argtypes = [C.POINTER(C.c_float), C.POINTER(_i32)]
_lib.lx_attn_set_rows_per_workgroup.argtypes = [_i32]
_lib.lx_ffn_set_token_tiles_per_workgroup.argtypes = [_i32]
_lib.lx_mlp_predict_mask.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _vp, _vp, _f, _vp, _vp]
_lib.lx_sparse_ffn_lora_fwd_workspace_bytes.restype = _sz
_lib.lx_sparse_ffn_lora_fwd_workspace_bytes.argtypes = [_i32, _i32]
_lib.lx_sparse_ffn_lora_bwd_workspace_bytes.restype = _sz
_lib.lx_sparse_ffn_lora_bwd_workspace_bytes.argtypes = [_i32, _i32, _i32, _i32]
_lib.lx_sparse_ffn_lora_fwd.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _i32, _vp, _vp, _vp, _vp, _vp,
                                        _blp, _vp, _vp, _vp, _vp, _sz, _vp]
_lib.lx_sparse_ffn_lora_bwd.argtypes = [C.c_int, _i32, _i32, _i32, _i32, _i32, _vp, _vp, _vp, _vp, _vp,
                                        _vp, _vp, _vp, _blp, _vp, _vp, _vp, _vp, _sz, _vp]
_lib.lx_attn_combine_patterns.argtypes = [_blp, _blp, _i32, _i32, _vp, _i32, _vp, _vp, _vp, _vp, _i32,
                                          _vp]


class LxError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {_lib.lx_status_string(status).decode()}")


def status_string(status: int) -> str:
    return _lib.lx_status_string(status).decode()


def _check(status: int, where: str):
    if status != LX_OK:
        raise LxError(status, where)


# The raw stream handle is read without building a torch.cuda.Stream object (2.9 us -> 0.3 us per call).
def _ptr(t):
    return None if t is None else t.data_ptr()


_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
_get_device = getattr(torch._C, "_cuda_getDevice", None)


def _stream():
    if _raw_stream is None or _get_device is None or not torch.cuda.is_initialized():
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_get_device())


_DTYPES = {torch.float32: LX_F32, torch.bfloat16: LX_BF16, torch.float16: LX_F16}


def _dt(t: torch.Tensor) -> int:
    dt = _DTYPES.get(t.dtype)
    if dt is None:
        raise LxError(LX_ERR_UNSUPPORTED, f"dtype {t.dtype}")
    return dt


class _ArgumentError(C.ArgumentError, TypeError):
    """An argument of a type that the C prototype does not take."""


def _convert(value, kind):
    """What a prototype with an argument of `kind` makes of a value that is no plain number."""
    if isinstance(value, kind):
        return value.value
    try:
        return kind(value).value
    except Exception:
        if hasattr(value, "_as_parameter_"):
            return _convert(value._as_parameter_, kind)
        raise _ArgumentError(f"{kind.__name__} expected, got {type(value).__name__}") from None


def _load_calls():
    """csrc/lx_call.cpp, bound to this module's library.  By path: it is this tree's."""
    loader = importlib.machinery.ExtensionFileLoader("_lx_call", CALL_PATH)
    m = importlib.util.module_from_spec(importlib.util.spec_from_loader("_lx_call", loader))
    loader.exec_module(m)
    m.bind({n: C.cast(getattr(_lib, n), _vp).value for n in EXPORTS}, _DTYPES, LxError, _stream,
           torch.uint8, torch.float32, torch.int32)
    m.types(lx_blocklist, _i32, _f, _convert, _ArgumentError)
    return m


_call = _load_calls()


class BlockList:
    """Device-resident row-compressed active-block list plus its host header."""

    def __init__(self, rows: int, cols: int, row_ptr: torch.Tensor, col_idx: torch.Tensor,
                 nnz_cap: int):
        self.rows, self.cols, self.nnz_cap = rows, cols, nnz_cap
        self.row_ptr, self.col_idx = row_ptr, col_idx
        self.c = lx_blocklist(rows, cols, row_ptr.data_ptr(), col_idx.data_ptr(), nnz_cap)
        self.ref = C.byref(self.c)   # made once: every call hands the same header over


def lx_mask_compact(mask: torch.Tensor, transpose: bool = False, nnz_cap: int | None = None,
                    out: BlockList | None = None) -> BlockList:
    """mask: uint8 device tensor [..., R, C]; leading dims are flattened into
    the list's rows.  transpose=True builds the column-compressed list."""
    if out is None:
        assert mask.dtype == torch.uint8 and mask.is_cuda and mask.is_contiguous() and mask.dim() >= 2
        rows, cols = (mask.shape[-1], mask.shape[-2]) if transpose else mask.shape[-2:]
        total = mask.numel() // cols
        cap = total * cols if nnz_cap is None else nnz_cap
        row_ptr = torch.empty(total + 1, dtype=torch.int32, device=mask.device)
        col_idx = torch.empty(max(cap, 1), dtype=torch.int32, device=mask.device)
        out = BlockList(total, cols, row_ptr, col_idx, cap)
    _call.mask_compact(mask, transpose, None if nnz_cap is None else max(nnz_cap, 1), out.row_ptr, out.col_idx)
    return out


def lx_mask_compact_pair(mask: torch.Tensor, out=None):
    """Row list and column list of the same masks [..., R, C] in one launch."""
    if out is None:
        assert mask.dtype == torch.uint8 and mask.is_cuda and mask.is_contiguous() and mask.dim() >= 2
        R, Cc = mask.shape[-2], mask.shape[-1]
        batch = mask.numel() // (R * Cc)
        cap = batch * R * Cc
        mk = lambda rows, cols: BlockList(
            batch * rows, cols, torch.empty(batch * rows + 1, dtype=torch.int32, device=mask.device),
            torch.empty(cap, dtype=torch.int32, device=mask.device), cap)
        out = (mk(R, Cc), mk(Cc, R))
    blr, blc = out
    _call.mask_compact_pair(mask, blr.row_ptr, blr.col_idx, blc.row_ptr, blc.col_idx)
    return blr, blc


class CompactBatch:
    """Pre-marshalled set of compaction jobs (up to 8) that run in one launch.
    add(mask, out, transpose) mirrors lx_mask_compact(mask, transpose, out=out)."""

    def __init__(self):
        self.jobs = []
        self._keep = []

    def add(self, mask: torch.Tensor, out: "BlockList", transpose: bool = False):
        assert mask.dtype == torch.uint8 and mask.is_cuda and mask.is_contiguous()
        R, Cc = mask.shape[-2], mask.shape[-1]
        batch = mask.numel() // (R * Cc)
        rows, cols, rs, cs = (Cc, R, 1, Cc) if transpose else (R, Cc, Cc, 1)
        assert out.rows == batch * rows and out.cols == cols
        self.jobs.append(lx_compact_job(mask.data_ptr(), batch, rows, cols, R * Cc, rs, cs,
                                        out.row_ptr.data_ptr(), out.col_idx.data_ptr(),
                                        out.col_idx.numel()))
        self._keep.append((mask, out))
        self._arr = (lx_compact_job * len(self.jobs))(*self.jobs)
        return self


def lx_mask_compact_batch(batch: CompactBatch):
    _check(_lib.lx_mask_compact_batch(batch._arr, len(batch.jobs), _stream()),
           "lx_mask_compact_batch")


def lx_attn_combine_patterns(pool_r: BlockList, pool_c: BlockList | None, nblk: int,
                             head_pattern: torch.Tensor, nnz_cap: int | None = None, out=None):
    """Multi-head list(s) from the pool layouts and the pattern id of every head.  Returns
    (row list, column list or None)."""
    Hm = head_pattern.numel()
    cap = Hm * nblk * nblk if nnz_cap is None else nnz_cap
    if out is None:
        assert head_pattern.dtype == torch.int32 and head_pattern.is_cuda and head_pattern.is_contiguous()
        mk = lambda: BlockList(Hm * nblk, nblk,
                               torch.empty(Hm * nblk + 1, dtype=torch.int32, device=head_pattern.device),
                               torch.empty(max(cap, 1), dtype=torch.int32, device=head_pattern.device), cap)
        out = (mk(), mk() if pool_c is not None else None)
    blr, blc = out
    _call.combine(pool_r.c, pool_c.c if pool_c is not None else None, pool_r.rows // nblk, nblk, head_pattern, max(cap, 1),
                  blr.row_ptr, blr.col_idx, blc.row_ptr if blc is not None else None,
                  blc.col_idx if blc is not None else None)
    return blr, blc


def lx_ffn_pack_weights(W_up: torch.Tensor, W_down: torch.Tensor):
    F, d = W_up.shape
    W_up_t = torch.empty((d, F), dtype=W_up.dtype, device=W_up.device)
    W_down_t = torch.empty((F, d), dtype=W_up.dtype, device=W_up.device)
    _check(_lib.lx_ffn_pack_weights(_dt(W_up), d, F, _ptr(W_up), _ptr(W_down), _ptr(W_up_t),
                                    _ptr(W_down_t), _stream()), "lx_ffn_pack_weights")
    return W_up_t, W_down_t


def lx_ffn_transpose(W: torch.Tensor, out: torch.Tensor | None = None) -> torch.Tensor:
    """[R,C] -> [C,R] on the device (one half of lx_ffn_pack_weights)."""
    R, Cc = W.shape
    if out is None:
        out = torch.empty((Cc, R), dtype=W.dtype, device=W.device)
    assert out.shape == (Cc, R) and out.is_contiguous()
    _check(_lib.lx_ffn_pack_weights(_dt(W), Cc, R, _ptr(W), None, _ptr(out), None, _stream()),
           "lx_ffn_pack_weights")
    return out


def lx_ffn_gather_weight_blocks(W: torch.Tensor, bl: BlockList, blk_n: int, out=None, compact=None):
    """W [F,d]: device tensor or pinned host tensor; bl: one-row device list.  Returns
    (Wc [nnz_cap*blk_n, d] on the device, one-row list of the compact matrix)."""
    assert W.dim() == 2 and W.is_contiguous()
    F, d = W.shape
    dev = bl.row_ptr.device
    if out is None:
        out = torch.zeros((bl.nnz_cap * blk_n, d), dtype=W.dtype, device=dev)
    if compact is None:
        compact = BlockList(1, bl.nnz_cap, torch.empty(2, dtype=torch.int32, device=dev),
                            torch.empty(bl.nnz_cap, dtype=torch.int32, device=dev), bl.nnz_cap)
    _check(_lib.lx_ffn_gather_weight_blocks(_dt(W), d, F, blk_n, _ptr(W), bl.ref, _ptr(out),
                                            _ptr(compact.row_ptr), _ptr(compact.col_idx), _stream()),
           "lx_ffn_gather_weight_blocks")
    return out, compact


def lx_sparse_ffn_fwd_workspace_bytes(dt, T, d, F, tile_t, blk_n, nnz_cap, have_h_act) -> int:
    return _lib.lx_sparse_ffn_fwd_workspace_bytes(dt, T, d, F, tile_t, blk_n, nnz_cap, have_h_act)


def lx_sparse_ffn_bwd_workspace_bytes(dt, T, d, F, tile_t, blk_n, nnz_cap, have_packed) -> int:
    return _lib.lx_sparse_ffn_bwd_workspace_bytes(dt, T, d, F, tile_t, blk_n, nnz_cap, have_packed)


def lx_sparse_ffn_split_workspace_bytes(dt, T, d, tile_t, bl: "BlockList") -> int:
    return _lib.lx_sparse_ffn_split_workspace_bytes(dt, T, d, tile_t, bl.ref)


def lx_sparse_ffn_lora_fwd_workspace_bytes(T, d) -> int:
    return _lib.lx_sparse_ffn_lora_fwd_workspace_bytes(T, d)


def lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, nnz_cap) -> int:
    return _lib.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, nnz_cap)


def lx_sparse_ffn_lora_fwd(X, W_up, A_pad, B_pad, W_down, bl: BlockList, Y, H_act, U, workspace=None):
    """U = X A_pad^T, H = ReLU(X W_up^T + U B_pad^T) on the listed blocks, Y = H W_down^T."""
    if workspace is None:
        T, d = X.shape
        workspace = torch.empty(_lib.lx_sparse_ffn_lora_fwd_workspace_bytes(T, d), dtype=torch.uint8,
                                device=X.device)
    _call.lora_fwd(X, W_up, A_pad, B_pad, W_down, bl.c, Y, H_act, U, workspace)


def lx_sparse_ffn_lora_bwd(X, dY, H_act, U, W_up_t, W_down_t, A_pad, B_pad, bl: BlockList, dX, dA, dB,
                           workspace):
    """dX, dA (fp32 [64,d]) and dB (fp32 [F,64]) of the LoRA-branch FFN."""
    _call.lora_bwd(X, dY, H_act, U, W_up_t, W_down_t, A_pad, B_pad, bl.c, dX, dA, dB, workspace)


def lx_mlp_predict_mask(X: torch.Tensor, Wa_t: torch.Tensor, thr: float, group_rows: int,
                        mask: torch.Tensor | None = None):
    """mask [T/group_rows, nblk] uint8 = OR over the tokens of a group of (X Wa_t^T > thr)."""
    if mask is None:
        mask = torch.empty((X.shape[0] // group_rows, Wa_t.shape[0]), dtype=torch.uint8, device=X.device)
    _call.predict(X, Wa_t, thr, group_rows, mask)
    return mask


def lx_sparse_attn_bwd_workspace_bytes(dt, B, Hh, S, D) -> int:
    return _lib.lx_sparse_attn_bwd_workspace_bytes(dt, B, Hh, S, D)


def lx_sparse_ffn_fwd(X, W_up, W_down, bl: BlockList, tile_t: int, blk_n: int, Y, H_act,
                      b_up=None, b_down=None, workspace=None):
    _call.ffn_fwd(X, W_up, W_down, bl.c, tile_t, blk_n, Y, H_act, b_up, b_down, workspace)
    return Y


def lx_sparse_ffn_bwd_dx(dY, H_act, W_up, W_down, bl: BlockList, tile_t: int, blk_n: int, dX,
                         workspace, W_up_t=None, W_down_t=None):
    _call.ffn_bwd(dY, H_act, W_up, W_down, bl.c, tile_t, blk_n, dX, workspace, W_up_t, W_down_t)
    return dX


def lx_profile_begin(kernel: int, max_launches: int):
    _check(_lib.lx_profile_begin(kernel, max_launches), "lx_profile_begin")


def lx_attn_set_rows_per_workgroup(rows: int):
    _check(_lib.lx_attn_set_rows_per_workgroup(rows), "lx_attn_set_rows_per_workgroup")


def lx_ffn_set_token_tiles_per_workgroup(tiles: int):
    _check(_lib.lx_ffn_set_token_tiles_per_workgroup(tiles), "lx_ffn_set_token_tiles_per_workgroup")


def lx_profile_end():
    """Returns (total kernel milliseconds, number of timed launches)."""
    ms, n = C.c_float(0), _i32(0)
    _check(_lib.lx_profile_end(C.byref(ms), C.byref(n)), "lx_profile_end")
    return ms.value, n.value


def lx_sparse_attn_fwd(Q, K, V, bl: BlockList, scale: float, causal: bool, O, LSE,
                       mask_batch: int = 1, head_active=None):
    _call.attn_fwd(Q, K, V, bl.c, scale, int(causal), O, LSE, mask_batch, head_active)
    return O, LSE


def lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, bl_rows: BlockList, bl_cols: BlockList,
                          scale: float, causal: bool, dQ, dK, dV, workspace, mask_batch: int = 1,
                          head_active=None):
    _call.attn_bwd(Q, K, V, O, LSE, dO, bl_rows.c, bl_cols.c, scale, int(causal), dQ, dK, dV, workspace, mask_batch,
                   head_active)
    return dQ, dK, dV


def lx_sparse_attn_bwd_dx_noalloc(Q, K, V, O, LSE, dO, bl_rows: BlockList, bl_cols: BlockList,
                                  scale: float, causal: bool, dQ, dK, dV, mask_batch: int = 1,
                                  head_active=None):
    _call.attn_bwd(Q, K, V, O, LSE, dO, bl_rows.c, bl_cols.c, scale, int(causal), dQ, dK, dV, mask_batch, head_active)
    return dQ, dK, dV


def lx_probe_mfma_rate(iters: int, sink: torch.Tensor) -> float:
    """Enqueues the MFMA rate probe; returns the FLOP of the launch."""
    fl = C.c_double(0.0)
    _check(_lib.lx_probe_mfma_rate(iters, _ptr(sink), C.byref(fl), _stream()), "lx_probe_mfma_rate")
    return fl.value


def lx_probe_stream_copy(src: torch.Tensor, dst: torch.Tensor) -> int:
    """Enqueues the stream-copy probe; returns the bytes moved (read + written)."""
    n = src.numel() * src.element_size()
    assert dst.numel() * dst.element_size() == n
    _check(_lib.lx_probe_stream_copy(_ptr(src), _ptr(dst), n, _stream()), "lx_probe_stream_copy")
    return 2 * n
