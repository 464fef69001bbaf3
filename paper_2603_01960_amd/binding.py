"""Python binding of libtiled_sdpa.so: argument marshalling only.

Every step of the forward pass runs in the HIP kernels behind the C-ABI declared
in include/tiled_sdpa.h.  PyTorch supplies device memory and the current stream.
The tensor functions (sdpa, sdpa_kv, sdpa_paged, sdpa_backward) go through native
code (csrc/torch_calls.cpp), the C-ABI itself is exposed through ctypes.
There is no CPU fallback: if the library is missing, loading raises.
"""
from __future__ import annotations

import ctypes
import math
from pathlib import Path

F16, BF16 = 0, 1
FLAG_LINEAR_GRID = 1
FLAG_EXACT_MAX = 2
FLAG_CAUSAL = 8

_PKG = Path(__file__).resolve().parent
_LIB_PATH = _PKG / "libtiled_sdpa.so"
_CALLS_PATH = _PKG / "_torch_calls.so"
_lib = None
_native = None

EXPORTS = (
    "tiled_sdpa_fwd",
    "tiled_sdpa_fwd_ex",
    "tiled_sdpa_bwd",
    "tiled_sdpa_bwd_gqa",
    "tiled_sdpa_bwd_workspace_bytes",
    "tiled_sdpa_bwd_full_workspace_bytes",
    "tiled_sdpa_default_tile",
    "tiled_sdpa_tune_tile",
    "tiled_sdpa_fwd_kv",
    "tiled_sdpa_fwd_gqa",
    "tiled_sdpa_fwd_kvcache",
    "tiled_sdpa_fwd_kvcache_static",
    "tiled_sdpa_fwd_paged",
    "tiled_sdpa_kv_default_splits",
    "tiled_sdpa_kv_tile_splits",
    "tiled_sdpa_kv_workspace_bytes",
    "tiled_sdpa_probe_mfma",
    "tiled_sdpa_probe_hbm_read",
    "tiled_sdpa_status_string",
    "tiled_sdpa_version",
)


class TiledSdpaError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"tiled_sdpa status {status}: {text}")
        self.status = status


def library_path() -> Path:
    return _LIB_PATH


def load_library():
    """Load the HIP library; raises if it has not been built (python -m paper_2603_01960_amd.build)."""
    global _lib
    if _lib is not None:
        return _lib
    if not _LIB_PATH.exists():
        raise FileNotFoundError(
            f"{_LIB_PATH} not found: build it with `python -m paper_2603_01960_amd.build` "
            "(there is no fallback path)")
    lib = ctypes.CDLL(str(_LIB_PATH))
    vp, ci, cf = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    lib.tiled_sdpa_fwd.restype = ci
    lib.tiled_sdpa_fwd.argtypes = [vp, vp, vp, vp, vp, ci, ci, ci, ci, cf, ci, vp]
    lib.tiled_sdpa_fwd_ex.restype = ci
    lib.tiled_sdpa_fwd_ex.argtypes = [vp, vp, vp, vp, vp, ci, ci, ci, ci, cf, ci, vp, ci, ci, ctypes.c_uint]
    lib.tiled_sdpa_default_tile.restype = ci
    lib.tiled_sdpa_default_tile.argtypes = [ci, ci, ci, ci, ci, ctypes.c_uint, ctypes.POINTER(ci), ctypes.POINTER(ci)]
    lib.tiled_sdpa_fwd_kv.restype = ci
    lib.tiled_sdpa_fwd_kv.argtypes = [vp, vp, vp, vp, vp, ci, ci, ci, ci, ci, cf, ci, vp, ci, ci, ctypes.c_uint,
                                      ci, vp, ctypes.c_ulonglong]
    lib.tiled_sdpa_kv_default_splits.restype = ci
    lib.tiled_sdpa_kv_default_splits.argtypes = [ci, ci, ci, ci, ci, ci, ctypes.c_uint, ctypes.POINTER(ci)]
    lib.tiled_sdpa_kv_tile_splits.restype = ci
    lib.tiled_sdpa_kv_tile_splits.argtypes = [ci, ci, ci, ci, ci, ci, ctypes.c_uint, ci, ci, ctypes.POINTER(ci)]
    lib.tiled_sdpa_kv_workspace_bytes.restype = ctypes.c_ulonglong
    lib.tiled_sdpa_kv_workspace_bytes.argtypes = [ci, ci, ci, ci, ci]
    lib.tiled_sdpa_bwd.restype = ci
    lib.tiled_sdpa_fwd_gqa.restype = ci
    lib.tiled_sdpa_fwd_gqa.argtypes = [vp] * 5 + [ci] * 6 + [cf, ci, vp, ci, ci, ctypes.c_uint, ci, vp, ctypes.c_ulonglong]
    lib.tiled_sdpa_fwd_kvcache.restype = ci
    lib.tiled_sdpa_fwd_kvcache.argtypes = [vp] * 6 + [ci] * 6 + [cf, ci, vp, ci, ci, ctypes.c_uint, ci, vp, ctypes.c_ulonglong]
    lib.tiled_sdpa_fwd_kvcache_static.restype = ci
    lib.tiled_sdpa_fwd_kvcache_static.argtypes = [vp] * 6 + [ci] * 6 + [cf, ci, vp, ci, ci, ctypes.c_uint, ci]
    lib.tiled_sdpa_fwd_paged.restype = ci
    lib.tiled_sdpa_fwd_paged.argtypes = [vp] * 7 + [ci] * 7 + [cf, ci, vp, ci, ci, ctypes.c_uint, ci, vp, ctypes.c_ulonglong]
    lib.tiled_sdpa_tune_tile.restype = ci
    lib.tiled_sdpa_tune_tile.argtypes = [vp] * 4 + [ci] * 4 + [cf, ci, vp, ctypes.c_uint, ci,
                                         ctypes.POINTER(ci), ctypes.POINTER(ci), ctypes.POINTER(cf)]
    lib.tiled_sdpa_bwd.argtypes = [vp] * 9 + [ci, ci, ci, ci, cf, ci, ctypes.c_uint, vp, ctypes.c_ulonglong, vp]
    lib.tiled_sdpa_bwd_gqa.restype = ci
    lib.tiled_sdpa_bwd_gqa.argtypes = [vp] * 9 + [ci, ci, ci, ci, ci, cf, ci, ctypes.c_uint, vp, ctypes.c_ulonglong, vp]
    lib.tiled_sdpa_bwd_workspace_bytes.restype = ctypes.c_ulonglong
    lib.tiled_sdpa_bwd_workspace_bytes.argtypes = [ci, ci, ci]
    lib.tiled_sdpa_bwd_full_workspace_bytes.restype = ctypes.c_ulonglong
    lib.tiled_sdpa_bwd_full_workspace_bytes.argtypes = [ci, ci, ci, ci, ci, ctypes.c_uint]
    lib.tiled_sdpa_probe_hbm_read.restype = ci
    lib.tiled_sdpa_probe_hbm_read.argtypes = [vp, ctypes.c_ulonglong, vp, ctypes.POINTER(ctypes.c_double), vp]
    lib.tiled_sdpa_probe_mfma.restype = ci
    lib.tiled_sdpa_probe_mfma.argtypes = [ci, ci, ci, vp, ctypes.POINTER(ctypes.c_double), vp]
    lib.tiled_sdpa_status_string.restype = ctypes.c_char_p
    lib.tiled_sdpa_status_string.argtypes = [ci]
    lib.tiled_sdpa_version.restype = ci
    lib.tiled_sdpa_version.argtypes = []
    _lib = lib
    return lib


def _calls():
    """The native tensor entry points (csrc/torch_calls.cpp)."""
    global _native
    if _native is None:
        import torch  # noqa: F401  (its libraries have to be in the process first)

        load_library()
        if not _CALLS_PATH.exists():
            raise FileNotFoundError(
                f"{_CALLS_PATH} not found: build it with `python -m paper_2603_01960_amd.build` "
                "(there is no fallback path)")
        from . import _torch_calls

        _native = _torch_calls
    return _native


def _checked(result):
    """Result object of a native call, or its status code as an exception."""
    if type(result) is int:
        raise TiledSdpaError(result, status_string(result))
    return result


def version() -> int:
    return int(load_library().tiled_sdpa_version())


def status_string(status: int) -> str:
    return load_library().tiled_sdpa_status_string(int(status)).decode()


TILE_ORDER = ((64, 32), (64, 64), (64, 128), (128, 32), (128, 64), (128, 128), (256, 64))


def tune_tile(q, k, v, causal: bool = False, scale=None, *, launches: int = 10, flags: int = 0):
    """Time every legal (T_M, T_N) on these tensors (tiled_sdpa_tune_tile; waits for the stream) and
    return ``((tile_m, tile_n), {tile: ms per launch})``.  Pass the tile to :func:`sdpa`."""
    import torch

    if causal:
        flags |= FLAG_CAUSAL
    for t in (q, k, v):
        if not isinstance(t, torch.Tensor) or not t.is_cuda or t.dim() != 4 or not t.is_contiguous():
            raise ValueError("q, k, v must be contiguous [B, H, S, D] device tensors")
    if q.dtype not in (torch.float16, torch.bfloat16) or k.dtype != q.dtype or v.dtype != q.dtype or \
            k.shape != q.shape or v.shape != q.shape:
        raise ValueError("q, k, v must share shape and dtype float16 or bfloat16")
    B, H, S, D = q.shape
    out = torch.empty_like(q)
    tm, tn = ctypes.c_int(0), ctypes.c_int(0)
    ms = (ctypes.c_float * len(TILE_ORDER))()
    with torch.cuda.device(q.device):
        stream = torch.cuda.current_stream(q.device).cuda_stream
        st = load_library().tiled_sdpa_tune_tile(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), B, H, S, D,
                                                 math.nan if scale is None else float(scale),
                                                 F16 if q.dtype == torch.float16 else BF16, stream, flags, launches,
                                                 ctypes.byref(tm), ctypes.byref(tn), ms)
    if st != 0:
        raise TiledSdpaError(st, status_string(st))
    return (tm.value, tn.value), {t: float(x) for t, x in zip(TILE_ORDER, ms) if x >= 0}


def default_tile(B: int, H: int, S: int, D: int, dtype: int, flags: int = 0):
    tm, tn = ctypes.c_int(0), ctypes.c_int(0)
    st = load_library().tiled_sdpa_default_tile(B, H, S, D, dtype, flags, ctypes.byref(tm), ctypes.byref(tn))
    if st != 0:
        raise TiledSdpaError(st, status_string(st))
    return tm.value, tn.value


def kv_default_splits(B: int, H: int, Sq: int, Skv: int, D: int, dtype: int, flags: int = 0) -> int:
    n = ctypes.c_int(0)
    st = load_library().tiled_sdpa_kv_default_splits(B, H, Sq, Skv, D, dtype, flags, ctypes.byref(n))
    if st != 0:
        raise TiledSdpaError(st, status_string(st))
    return n.value


def kv_workspace_bytes(B: int, H: int, Sq: int, D: int, splits: int) -> int:
    return int(load_library().tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits))


def probe_mfma(dtype: int, random_operands, iters: int, sink=None, stream=None) -> float:
    """Enqueue the MFMA stream (see tiled_sdpa_probe_mfma); returns its flop count.

    ``random_operands``: False/0 constant operands, True/1 random ones, 2 random ones plus the
    attention loop's LDS-read and vector-ALU mix.

    With ``iters=0`` nothing is launched (flop count only) and ``sink`` may be None; a launch
    (``iters > 0``) needs a real device buffer of 512*256 floats."""
    if sink is None and iters != 0:
        raise ValueError("probe_mfma: iters > 0 launches a kernel that writes 512*256 floats to `sink`")
    flops = ctypes.c_double(0.0)
    st = load_library().tiled_sdpa_probe_mfma(dtype, int(random_operands), iters, sink, ctypes.byref(flops), stream)
    if st != 0:
        raise TiledSdpaError(st, status_string(st))
    return flops.value


def probe_hbm_read(src_ptr: int, nbytes: int, sink_ptr: int, stream=None) -> float:
    """Enqueue the read-only stream over ``nbytes`` at ``src_ptr`` (see tiled_sdpa_probe_hbm_read); returns
    the bytes it reads."""
    done = ctypes.c_double(0.0)
    st = load_library().tiled_sdpa_probe_hbm_read(src_ptr, nbytes, sink_ptr, ctypes.byref(done), stream)
    if st != 0:
        raise TiledSdpaError(st, status_string(st))
    return done.value


def tiled_sdpa_fwd(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, S, D, scale, dtype, stream) -> int:
    """Raw call: integer device addresses in, status code out (same argument order as the C-ABI)."""
    return int(load_library().tiled_sdpa_fwd(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, S, D,
                                             float(scale), dtype, stream))


def tiled_sdpa_fwd_ex(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, S, D, scale, dtype, stream,
                      tile_m=0, tile_n=0, flags=0) -> int:
    return int(load_library().tiled_sdpa_fwd_ex(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, S, D,
                                                float(scale), dtype, stream, tile_m, tile_n, flags))


def tiled_sdpa_fwd_kv(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, Sq, Skv, D, scale, dtype, stream,
                      tile_m=0, tile_n=0, flags=0, splits=0, workspace_ptr=None, workspace_bytes=0) -> int:
    return int(load_library().tiled_sdpa_fwd_kv(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, Sq, Skv, D,
                                                float(scale), dtype, stream, tile_m, tile_n, flags,
                                                splits, workspace_ptr, workspace_bytes))


def tiled_sdpa_fwd_gqa(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, Hkv, Sq, Skv, D, scale, dtype, stream,
                       tile_m=0, tile_n=0, flags=0, splits=0, workspace_ptr=None, workspace_bytes=0) -> int:
    return int(load_library().tiled_sdpa_fwd_gqa(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, B, H, Hkv, Sq, Skv, D,
                                                 float(scale), dtype, stream, tile_m, tile_n, flags,
                                                 splits, workspace_ptr, workspace_bytes))


def tiled_sdpa_fwd_kvcache(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, kv_lens_ptr, B, H, Hkv, Sq, Skv, D, scale, dtype,
                           stream, tile_m=0, tile_n=0, flags=0, splits=0, workspace_ptr=None, workspace_bytes=0) -> int:
    return int(load_library().tiled_sdpa_fwd_kvcache(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, kv_lens_ptr, B, H, Hkv, Sq,
                                                     Skv, D, float(scale), dtype, stream, tile_m, tile_n, flags,
                                                     splits, workspace_ptr, workspace_bytes))


STATIC_SCRATCH_BYTES = 32 * 1024 * 1024


def tiled_sdpa_fwd_kvcache_static(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, kv_lens_ptr, B, H, Hkv, Sq, Skv, D, scale, dtype,
                                  stream, tile_m=0, tile_n=0, flags=0, splits=0) -> int:
    """tiled_sdpa_fwd_kvcache with the split states in the library's own static device buffer."""
    return int(load_library().tiled_sdpa_fwd_kvcache_static(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, kv_lens_ptr, B, H, Hkv,
                                                            Sq, Skv, D, float(scale), dtype, stream, tile_m, tile_n,
                                                            flags, splits))


def sdpa_kv(q, k, v, causal: bool = False, scale=None, *, splits: int = 0, return_lse: bool = False,
            out=None, workspace=None, tile=None, flags: int = 0, kv_lens=None):
    """Attention of q [B, H, Sq, D] over k, v [B, H, Skv, D] (KV-cache / decoding shapes), the key range
    split over ``splits`` workgroups per query tile (0 = heuristic).  Under ``causal`` the queries are
    the last Sq positions of the sequence.  ``workspace`` (any dense tensor of enough bytes on q's device)
    is allocated through torch when not given and needed.

    Grouped heads: k, v may be [B, Hkv, Skv, D] with H = G * Hkv, query head h reading key/value head
    h // G (tiled_sdpa_fwd_gqa): the rows of a group share one pass over its keys.

    ``kv_lens`` (int32 device tensor [B]): k, v are a cache of capacity Skv of which batch entry b holds
    kv_lens[b] valid rows (tiled_sdpa_fwd_kvcache); rows no key reaches come back as zeros.
    """
    return _checked(_calls().sdpa_kv(q, k, v, causal, scale, splits, return_lse, out, workspace, tile, flags, kv_lens))


def tiled_sdpa_fwd_paged(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, kv_lens_ptr, block_table_ptr, B, H, Hkv, Sq, max_blocks,
                         block_rows, D, scale, dtype, stream, tile_m=0, tile_n=0, flags=0, splits=0,
                         workspace_ptr=None, workspace_bytes=0) -> int:
    return int(load_library().tiled_sdpa_fwd_paged(q_ptr, k_ptr, v_ptr, o_ptr, lse_ptr, kv_lens_ptr, block_table_ptr,
                                                   B, H, Hkv, Sq, max_blocks, block_rows, D, float(scale), dtype,
                                                   stream, tile_m, tile_n, flags, splits, workspace_ptr, workspace_bytes))


def sdpa_paged(q, k_pages, v_pages, kv_lens, block_table, causal: bool = False, scale=None, *, splits: int = 0,
               return_lse: bool = False, out=None, workspace=None, tile=None, flags: int = 0):
    """Attention of q [B, H, Sq, D] over a paged cache: k_pages, v_pages [P, Hkv, block_rows, D],
    block_table int32 [B, max_blocks] (page of every block of every batch entry), kv_lens int32 [B]
    (valid key rows per entry).  See tiled_sdpa_fwd_paged; otherwise as :func:`sdpa_kv`."""
    return _checked(_calls().sdpa_paged(q, k_pages, v_pages, kv_lens, block_table, causal, scale, splits, return_lse, out,
                                        workspace, tile, flags))


def bwd_workspace_bytes(B: int, H: int, S: int) -> int:
    return int(load_library().tiled_sdpa_bwd_workspace_bytes(B, H, S))


def bwd_full_workspace_bytes(B: int, H: int, Hkv: int, S: int, D: int, causal: bool = False) -> int:
    """Workspace with which the backward pass is fastest; see tiled_sdpa_bwd_full_workspace_bytes."""
    return int(load_library().tiled_sdpa_bwd_full_workspace_bytes(B, H, Hkv, S, D, FLAG_CAUSAL if causal else 0))


def tiled_sdpa_bwd(q_ptr, k_ptr, v_ptr, o_ptr, dout_ptr, lse_ptr, dq_ptr, dk_ptr, dv_ptr, B, H, S, D, scale,
                   dtype, flags, workspace_ptr, workspace_bytes, stream) -> int:
    return int(load_library().tiled_sdpa_bwd(q_ptr, k_ptr, v_ptr, o_ptr, dout_ptr, lse_ptr, dq_ptr, dk_ptr,
                                             dv_ptr, B, H, S, D, float(scale), dtype, flags,
                                             workspace_ptr, workspace_bytes, stream))


def sdpa_backward(q, k, v, o, dout, lse, causal: bool = False, scale=None, *, workspace=None, grads=None):
    """(dq, dk, dv) for the attention of :func:`sdpa`; ``o`` and ``lse`` are that call's outputs
    (``return_lse=True``) for the same q, k, v, causal and scale.  ``grads=(dq, dk, dv)`` and
    ``workspace`` let the caller own the buffers; otherwise torch allocates them.

    The workspace that torch allocates is :func:`bwd_full_workspace_bytes`: for large calls at D = 64, 96 and 128 FP32 sums of dQ, twice
    the bytes of q and at most 2.3 GB (in a captured graph they stay with the graph).  If it cannot be had, and with a caller's workspace of at
    least :func:`bwd_workspace_bytes` but less than that, the call takes kernels without such sums: 0.9 of the speed, the gradients differ
    in their last bits.  The same workspace size always gives the same bits; a program that needs them to not depend on
    the memory that is free passes a workspace.

    Grouped heads: k, v [B, Hkv, S, D] with H a multiple of Hkv (the forward of ``sdpa_kv`` at Sq = Skv);
    dk, dv then have the shape of k and hold the sum over the query heads of each group."""
    return _checked(_calls().sdpa_backward(q, k, v, o, dout, lse, causal, scale, workspace, grads))


def sdpa(q, k, v, causal: bool = False, scale=None, *, return_lse: bool = False, out=None,
         lse_out=None, tile=None, flags: int = 0):
    """o = softmax(q k^T * scale [+ causal mask]) v for contiguous [B, H, S, D] FP16/BF16 device tensors.

    Mirrors the functional API of Section 4.2.1 of the paper (scale defaults to 1/sqrt(D)).
    ``tile=(T_M, T_N)`` pins the schedule; ``out`` / ``lse_out`` let the caller own the outputs.
    """
    return _checked(_calls().sdpa(q, k, v, causal, scale, return_lse, out, lse_out, tile, flags))
