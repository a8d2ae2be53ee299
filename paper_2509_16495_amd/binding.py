"""Thin Python binding of the C ABI in include/shiftattn.h.

Argument marshalling only: every function takes torch tensors that already live on the GPU,
checks shapes, and passes raw device pointers plus the current HIP stream to libshiftattn.so.
All of the path's work happens in the library's kernels; there is no Python or CPU fallback.
If the library has not been built (python -m paper_2509_16495_amd.build, or
__graft_entry__.build()), loading raises.
"""
from __future__ import annotations

import ctypes
import importlib
import os
from typing import Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# The variable names another build of the library, of the same interface (include/shiftattn.h); the calls are always the package's.
LIB_PATH = os.environ.get("SHIFTATTN_LIB") or os.path.join(_HERE, "libshiftattn.so")
CALLS_PATH = os.path.join(_HERE, "_calls.so")

OK, EINVAL, EUNSUPPORTED, EWORKSPACE, EHIP = 0, -1, -2, -3, -4
BF16, F32 = 0, 1
BLOCK_SIZE = 16


class ShiftAttnError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"shiftattn error {code}: {msg}")
        self.code = code


class Xchg(ctypes.Structure):
    _fields_ = [("P", ctypes.c_int32), ("num_q_heads", ctypes.c_int32), ("num_kv_heads", ctypes.c_int32),
                ("head_dim", ctypes.c_int32), ("dtype", ctypes.c_int32)]


class Attn(ctypes.Structure):
    _fields_ = [("num_q_heads", ctypes.c_int32), ("num_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("dtype", ctypes.c_int32), ("block_size", ctypes.c_int32), ("num_blocks", ctypes.c_int32),
                ("max_blocks_per_seq", ctypes.c_int32), ("softmax_scale", ctypes.c_float),
                ("q_stride", ctypes.c_int64), ("kv_stride", ctypes.c_int64), ("out_stride", ctypes.c_int64),
                ("kv_format", ctypes.c_int32), ("k_scale", ctypes.c_float), ("v_scale", ctypes.c_float),
                ("reserved", ctypes.c_int32)]


class PrefillPlan(ctypes.Structure):
    _fields_ = [("tile_columns", ctypes.c_int32), ("wave_columns", ctypes.c_int32), ("key_ranges", ctypes.c_int32),
                ("tiles_per_wg", ctypes.c_int32), ("decode_wgs", ctypes.c_int32)]


class ProjPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("streams", "k_ranges", "token_pieces", "feature_pieces", "lead_tiles", "lead_features",
                                              "lead_tokens", "tile_features", "tile_tokens")]


KV_SAME, KV_FP8_E4M3 = 0, 1


_lib: Optional[ctypes.CDLL] = None
_calls = None  # csrc/python_calls.cpp, bound to _lib


def is_built() -> bool:
    return os.path.exists(LIB_PATH) and os.path.exists(CALLS_PATH)


def _workspace(need: int, like: torch.Tensor) -> torch.Tensor:
    return torch.empty(need, dtype=torch.uint8, device=like.device)


def lib() -> ctypes.CDLL:
    """The loaded C library.  Raises if it was never built: there is no other implementation."""
    global _lib, _calls
    if _lib is None:
        for path in (LIB_PATH, CALLS_PATH):
            if not os.path.exists(path):
                raise RuntimeError(f"{path} is missing: build it with `python -m paper_2509_16495_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        vp, i32, i64p, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_size_t
        xp, ap = ctypes.POINTER(Xchg), ctypes.POINTER(Attn)
        L.shiftattn_pack_seq2head.argtypes = [vp, vp, i32, i32, xp, vp]
        L.shiftattn_unpack_head2seq.argtypes = [vp, vp, i32, i32, xp, vp]
        L.shiftattn_qkv_proj_pack.argtypes = [vp, vp, vp, i32, i32, i32, xp, vp]
        L.shiftattn_unpack_o_proj.argtypes = [vp, vp, vp, i32, i32, i32, xp, vp]
        L.shiftattn_qkv_proj_pack_ws.argtypes = [vp, vp, vp, i32, i32, i32, xp, vp, ctypes.c_size_t, vp]
        L.shiftattn_unpack_o_proj_ws.argtypes = [vp, vp, vp, i32, i32, i32, xp, vp, ctypes.c_size_t, vp]
        L.shiftattn_proj_workspace_bytes.argtypes = [i32, i32, i32]
        L.shiftattn_proj_workspace_bytes.restype = ctypes.c_size_t
        L.shiftattn_proj_workspace_bytes_fp8.argtypes = [i32, i32, i32]
        L.shiftattn_proj_workspace_bytes_fp8.restype = ctypes.c_size_t
        L.shiftattn_qkv_proj_pack_fp8_ws.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, xp, vp, ctypes.c_size_t, vp]
        L.shiftattn_unpack_o_proj_fp8_ws.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, xp, vp, ctypes.c_size_t, vp]
        L.shiftattn_quantize_rows_fp8.argtypes = [vp, vp, vp, i32, i32, vp]
        L.shiftattn_quantize_recv_fp8.argtypes = [vp, vp, vp, i32, i32, xp, vp]
        L.shiftattn_qkv_proj_pack_fp8.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, xp, vp]
        L.shiftattn_unpack_o_proj_fp8.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, xp, vp]
        L.shiftattn_kv_write.argtypes = [vp, vp, i64p, i32, vp, ap, vp]
        L.shiftattn_prefill.argtypes = [vp, vp, vp, i64p, vp, vp, vp, vp, i32, i32, i32, i32, vp, vp, sz, ap, vp]
        L.shiftattn_decode.argtypes = [vp, vp, vp, i64p, vp, vp, vp, i32, i32, vp, vp, sz, ap, vp]
        L.shiftattn_decode_static.argtypes = [vp, vp, vp, i64p, vp, vp, vp, i32, i32, vp, ap, vp]
        L.shiftattn_prefill_workspace_bytes.argtypes = [i32, i32, i32, i32, ap]
        L.shiftattn_prefill_workspace_bytes.restype = sz
        L.shiftattn_decode_workspace_bytes.argtypes = [i32, i32, ap]
        L.shiftattn_decode_workspace_bytes.restype = sz
        L.shiftattn_mixed.argtypes = [vp, vp, vp, i64p, vp, vp, vp, vp, i32, i32, i32, i32, i32, i32, vp, vp, sz, ap, vp]
        L.shiftattn_mixed_workspace_bytes.argtypes = [i32, i32, i32, i32, i32, i32, ap]
        L.shiftattn_mixed_workspace_bytes.restype = sz
        L.shiftattn_head_block.argtypes = [i32, i32, i32]
        L.shiftattn_head_block.restype = i32
        L.shiftattn_kv_head_of_block.argtypes = [i32, i32, i32]
        L.shiftattn_kv_head_of_block.restype = i32
        L.shiftattn_padded_tokens.argtypes = [i32, i32]
        L.shiftattn_padded_tokens.restype = i32
        L.shiftattn_use_base_config.argtypes = [i32, i32]
        L.shiftattn_use_base_config.restype = i32
        L.shiftattn_ceiling_mfma_bf16.argtypes = [vp, vp, i32, ctypes.POINTER(ctypes.c_int64), vp]
        L.shiftattn_ceiling_mfma_bf16_fresh.argtypes = [vp, vp, i32, ctypes.POINTER(ctypes.c_int64), vp]
        L.shiftattn_ceiling_hbm_read.argtypes = [vp, sz, vp, ctypes.POINTER(ctypes.c_int64), vp]
        L.shiftattn_ceiling_hbm_copy.argtypes = [vp, vp, sz, ctypes.POINTER(ctypes.c_int64), vp]
        L.shiftattn_set_option.argtypes = [i32, i32]
        L.shiftattn_get_option.argtypes = [i32]
        L.shiftattn_get_option.restype = i32
        L.shiftattn_last_error.restype = ctypes.c_char_p
        _calls = importlib.import_module("._calls", __package__)
        _calls.bind(_workspace, *[ctypes.cast(getattr(L, name), ctypes.c_void_p).value for name in _calls.names])
        _lib = L
    return _lib


OPT_PREFILL_TILE, OPT_PREFILL_SPLITS, OPT_GENERIC_ONLY, OPT_PREFILL_PAIRING, OPT_PREFILL_SCALED_Q = 0, 1, 2, 3, 4


def init() -> None:
    _check(lib().shiftattn_init())


def set_option(option: int, value: int) -> None:
    _check(lib().shiftattn_set_option(option, value))


def get_option(option: int) -> int:
    return int(lib().shiftattn_get_option(option))


def last_error() -> str:
    return lib().shiftattn_last_error().decode()


def _check(rc: int) -> None:
    if rc != OK:
        raise ShiftAttnError(rc, last_error())


# Small calls are bound by what the host does per launch, so the functions of the path hand their arguments to
# csrc/python_calls.cpp, which checks them and calls the library, and asks for a workspace only where a call brings none
# (the library checks the size by itself).
def _native():
    if _lib is None:
        lib()
    return _calls


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else t.data_ptr()


if hasattr(torch._C, "_cuda_getCurrentRawStream"):
    def _stream() -> int:
        return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())
else:
    def _stream() -> int:
        return torch.cuda.current_stream().cuda_stream


# ---- host-only helpers --------------------------------------------------------------------------
def head_block(sp: int, tp: int, rank: int) -> int:
    return int(lib().shiftattn_head_block(sp, tp, rank))


def kv_head_of_block(block: int, P: int, h_kv: int) -> int:
    return int(lib().shiftattn_kv_head_of_block(block, P, h_kv))


def padded_tokens(n: int, sp: int) -> int:
    return int(lib().shiftattn_padded_tokens(n, sp))


def use_base_config(n_tokens: int, threshold: int) -> int:
    return int(lib().shiftattn_use_base_config(n_tokens, threshold))


def prefill_plan(num_seqs: int, total_q: int, max_q_len: int, max_seq_len: int, desc: Attn, num_decode_seqs: int = 0,
                 max_decode_seq_len: int = 0) -> PrefillPlan:
    """The launch that such a prefill call, or such a unified batch's chunks, takes (host only)."""
    plan = PrefillPlan()
    query = lib().shiftattn_prefill_plan
    query.argtypes = [ctypes.c_int32] * 6 + [ctypes.POINTER(Attn), ctypes.POINTER(PrefillPlan)]
    _check(query(num_seqs, total_q, max_q_len, max_seq_len, num_decode_seqs, max_decode_seq_len, ctypes.byref(desc), ctypes.byref(plan)))
    return plan


def proj_plan(rows: int, n_features: int, k: int, fp8: bool = False, workspace_bytes: Optional[int] = None) -> ProjPlan:
    """The launch that a projection of `rows` token rows with an [n_features, k] matrix takes (host only); workspace_bytes
    None: with the workspace that the size query names."""
    plan = ProjPlan()
    query = lib().shiftattn_proj_plan
    query.argtypes = [ctypes.c_int32] * 4 + [ctypes.c_size_t, ctypes.POINTER(ProjPlan)]
    given = proj_workspace_bytes(rows, n_features, k, fp8) if workspace_bytes is None else workspace_bytes
    _check(query(rows, n_features, k, int(fp8), given, ctypes.byref(plan)))
    return plan


def ceiling_mfma_bf16(operands: torch.Tensor, sink: torch.Tensor, iters: int) -> int:
    """Enqueue the MFMA-only probe; returns the flops of the launch."""
    assert operands.numel() * operands.element_size() >= 2048 and operands.is_contiguous()
    flops = ctypes.c_int64(0)
    _check(lib().shiftattn_ceiling_mfma_bf16(_ptr(operands), _ptr(sink), iters, ctypes.byref(flops), _stream()))
    return flops.value


def ceiling_mfma_bf16_fresh(operands: torch.Tensor, sink: torch.Tensor, iters: int) -> int:
    """Enqueue the MFMA-only probe whose operands change from one MFMA to the next; returns the flops of the launch."""
    assert operands.numel() * operands.element_size() >= 16384 and operands.is_contiguous()
    flops = ctypes.c_int64(0)
    _check(lib().shiftattn_ceiling_mfma_bf16_fresh(_ptr(operands), _ptr(sink), iters, ctypes.byref(flops), _stream()))
    return flops.value


def copy_probe(src: torch.Tensor, dst: torch.Tensor) -> int:
    """Enqueue the read + write streaming probe over all of `src`; returns the bytes copied."""
    assert src.is_contiguous() and dst.is_contiguous() and dst.numel() * dst.element_size() >= src.numel() * src.element_size()
    n = ctypes.c_int64(0)
    _check(lib().shiftattn_ceiling_hbm_copy(_ptr(src), _ptr(dst), src.numel() * src.element_size(), ctypes.byref(n), _stream()))
    return n.value


def ceiling_hbm_read(src: torch.Tensor, sink: torch.Tensor) -> int:
    """Enqueue the streaming-read probe over all of `src`; returns the bytes requested."""
    assert src.is_contiguous()
    n = ctypes.c_int64(0)
    _check(lib().shiftattn_ceiling_hbm_read(_ptr(src), src.numel() * src.element_size(), _ptr(sink), ctypes.byref(n),
                                            _stream()))
    return n.value


def local_kv_heads(P: int, h_kv: int) -> int:
    return 0 if h_kv == 0 else (h_kv // P if h_kv >= P else 1)


# ---- exchange pack / unpack -----------------------------------------------------------------------
def pack_seq2head(qkv: torch.Tensor, send: torch.Tensor, P: int, h: int, h_kv: int) -> None:
    """qkv [T, h+2*h_kv, D] -> send [P, T_pad, h/P + 2*hkv_l, D] (pad rows zeroed)."""
    _check(_native().pack_seq2head(qkv, send, P, h, h_kv))


def unpack_head2seq(recv: torch.Tensor, out: torch.Tensor) -> None:
    """recv [P, T_pad, h/P, D] -> out [T, h, D]."""
    _check(_native().unpack_head2seq(recv, out))


# ---- KV cache and attention -------------------------------------------------------------------------
def proj_workspace_bytes(rows: int, n_features: int, k: int, fp8: bool = False) -> int:
    """Bytes of workspace that a projection of `rows` token rows with an [n_features, k] matrix makes good use of (or more than it uses)."""
    if fp8:
        return int(lib().shiftattn_proj_workspace_bytes_fp8(rows, n_features, k))
    return int(lib().shiftattn_proj_workspace_bytes(rows, n_features, k))


def qkv_proj_pack(x: torch.Tensor, w_qkv: torch.Tensor, send: torch.Tensor, P: int, h: int, h_kv: int,
                  workspace: Optional[torch.Tensor] = None) -> None:
    """x [T, d_model], w_qkv [(h + 2 h_kv) D, d_model] -> send [P, T_pad, hq_l + 2 hkv_l, D] (projection + pack)."""
    _check(_native().qkv_proj_pack(x, w_qkv, send, P, h, h_kv, workspace))


def unpack_o_proj(recv: torch.Tensor, w_o: torch.Tensor, out: torch.Tensor, workspace: Optional[torch.Tensor] = None) -> None:
    """recv [P, T_pad, hq_l, D], w_o [d_model, h D] -> out [T, d_model] (unpack + projection)."""
    _check(_native().unpack_o_proj(recv, w_o, out, workspace))


def quantize_rows_fp8(x: torch.Tensor, codes: torch.Tensor, scales: torch.Tensor) -> None:
    """x [rows, cols] bf16 -> codes [rows, cols] uint8 (FP8 E4M3), scales [rows] float32 (amax / 448)."""
    _check(_native().quantize_rows_fp8(x, codes, scales))


def quantize_recv_fp8(recv: torch.Tensor, codes: torch.Tensor, scales: torch.Tensor) -> None:
    """recv [P, T_pad, hq_l, D] bf16 -> codes of the same shape (uint8), scales [T]: one scale per token over all buffers."""
    _check(_native().quantize_recv_fp8(recv, codes, scales))


def qkv_proj_pack_fp8(x_codes: torch.Tensor, x_scales: torch.Tensor, w_codes: torch.Tensor, w_scales: torch.Tensor,
                      send: torch.Tensor, P: int, h: int, h_kv: int, workspace: Optional[torch.Tensor] = None) -> None:
    """FP8 E4M3 codes x [T, d_model] and w [(h + 2 h_kv) D, d_model] with their row scales -> bf16 send buffers."""
    _check(_native().qkv_proj_pack_fp8(x_codes, x_scales, w_codes, w_scales, send, P, h, h_kv, workspace))


def unpack_o_proj_fp8(recv_codes: torch.Tensor, a_scales: torch.Tensor, w_codes: torch.Tensor, w_scales: torch.Tensor,
                      out: torch.Tensor, workspace: Optional[torch.Tensor] = None) -> None:
    """FP8 E4M3 codes recv [P, T_pad, hq_l, D] (one scale per token) and w [d_model, h D] (one per feature) -> out [T, d_model] bf16."""
    _check(_native().unpack_o_proj_fp8(recv_codes, a_scales, w_codes, w_scales, out, workspace))


def attn_desc(q: torch.Tensor, kv_cache: torch.Tensor, block_table: torch.Tensor, softmax_scale: float,
              k_new: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None, k_scale: float = 1.0,
              v_scale: float = 1.0) -> Attn:
    """Descriptor from tensor shapes.  kv_cache is [num_blocks, hkv_l, 2, 16*D] in q's type, or uint8 for an
    FP8 E4M3 cache (then k_scale / v_scale give the value of a code)."""
    return Attn.from_buffer_copy(_native().attn_desc(q, kv_cache, block_table, softmax_scale, k_new, out, k_scale, v_scale))


def kv_write(k_new: torch.Tensor, v_new: torch.Tensor, slot_mapping: torch.Tensor, kv_cache: torch.Tensor,
             k_scale: float = 1.0, v_scale: float = 1.0) -> None:
    _check(_native().kv_write(k_new, v_new, slot_mapping, kv_cache, k_scale, v_scale))


def prefill_workspace_bytes(num_seqs: int, total_q: int, max_q_len: int, max_seq_len: int, a: Attn) -> int:
    return int(lib().shiftattn_prefill_workspace_bytes(num_seqs, total_q, max_q_len, max_seq_len, ctypes.byref(a)))


def decode_workspace_bytes(num_seqs: int, max_seq_len: int, a: Attn) -> int:
    return int(lib().shiftattn_decode_workspace_bytes(num_seqs, max_seq_len, ctypes.byref(a)))


def prefill(q: torch.Tensor, kv_cache: torch.Tensor, block_table: torch.Tensor, cu_seqlens_q: torch.Tensor,
            seq_lens: torch.Tensor, max_q_len: int, max_seq_len: int, out: torch.Tensor, softmax_scale: float,
            k_new: Optional[torch.Tensor] = None, v_new: Optional[torch.Tensor] = None,
            slot_mapping: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None, k_scale: float = 1.0,
            v_scale: float = 1.0) -> None:
    """Causal attention of prefill chunks; q/out [total_q, hq_l, D] (row-strided views allowed)."""
    _check(_native().prefill(q, kv_cache, block_table, cu_seqlens_q, seq_lens, max_q_len, max_seq_len, out, softmax_scale, k_new, v_new,
                             slot_mapping, workspace, k_scale, v_scale))


def decode(q: torch.Tensor, kv_cache: torch.Tensor, block_table: torch.Tensor, seq_lens: torch.Tensor,
           max_seq_len: int, out: torch.Tensor, softmax_scale: float, k_new: Optional[torch.Tensor] = None,
           v_new: Optional[torch.Tensor] = None, slot_mapping: Optional[torch.Tensor] = None,
           workspace: Optional[torch.Tensor] = None, k_scale: float = 1.0, v_scale: float = 1.0) -> None:
    """One new token per sequence; q/out [num_seqs, hq_l, D]."""
    _check(_native().decode(q, kv_cache, block_table, seq_lens, max_seq_len, out, softmax_scale, k_new, v_new, slot_mapping, workspace,
                            k_scale, v_scale))


STATIC_SCRATCH_BYTES = 16 << 20


def decode_static(q: torch.Tensor, kv_cache: torch.Tensor, block_table: torch.Tensor, seq_lens: torch.Tensor,
                  max_seq_len: int, out: torch.Tensor, softmax_scale: float, k_new: Optional[torch.Tensor] = None,
                  v_new: Optional[torch.Tensor] = None, slot_mapping: Optional[torch.Tensor] = None, k_scale: float = 1.0,
                  v_scale: float = 1.0) -> None:
    """decode() without a workspace: the library's own static device array takes the split partials."""
    _check(_native().decode_static(q, kv_cache, block_table, seq_lens, max_seq_len, out, softmax_scale, k_new, v_new, slot_mapping, None,
                                   k_scale, v_scale))


def mixed_workspace_bytes(num_prefill_seqs: int, total_prefill_q: int, max_q_len: int, max_prefill_seq_len: int,
                          num_decode_seqs: int, max_decode_seq_len: int, a: Attn) -> int:
    return int(lib().shiftattn_mixed_workspace_bytes(num_prefill_seqs, total_prefill_q, max_q_len, max_prefill_seq_len,
                                                     num_decode_seqs, max_decode_seq_len, ctypes.byref(a)))


def mixed(q: torch.Tensor, kv_cache: torch.Tensor, block_table: torch.Tensor, cu_seqlens_q: torch.Tensor,
          seq_lens: torch.Tensor, num_prefill_seqs: int, max_q_len: int, max_prefill_seq_len: int,
          max_decode_seq_len: int, out: torch.Tensor, softmax_scale: float, k_new: Optional[torch.Tensor] = None,
          v_new: Optional[torch.Tensor] = None, slot_mapping: Optional[torch.Tensor] = None,
          workspace: Optional[torch.Tensor] = None, k_scale: float = 1.0, v_scale: float = 1.0) -> None:
    """Unified batch: the first num_prefill_seqs sequences are chunks (cu_seqlens_q [num_prefill_seqs + 1]), the
    others carry one row each; q/out hold the chunk rows first, then the decode rows."""
    _check(_native().mixed(q, kv_cache, block_table, cu_seqlens_q, seq_lens, num_prefill_seqs, max_q_len, max_prefill_seq_len,
                           max_decode_seq_len, out, softmax_scale, k_new, v_new, slot_mapping, workspace, k_scale, v_scale))


# ---- numpy <-> device helpers for tests and benchmarks (storage only) ------------------------------------
def to_device(a, dtype: str, device: str = "cuda:0") -> torch.Tensor:
    """numpy array in the workloads storage convention (uint16 bit patterns for bf16) -> GPU tensor."""
    import numpy as np
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(device)
    return torch.from_numpy(np.ascontiguousarray(a)).to(device)


def to_host(t: torch.Tensor):
    """GPU tensor -> numpy array in the workloads storage convention."""
    import numpy as np
    t = t.detach().contiguous().cpu()
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).numpy().view(np.uint16)
    return t.numpy()
