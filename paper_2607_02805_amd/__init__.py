"""Python binding of libbdlm, the MI355X (gfx950) block-restricted bidirectional Mamba scan.

Argument marshalling only: every step of the computation runs in the HIP kernels
behind the C ABI declared in ``include/bdlm.h``.  PyTorch supplies device memory
and the stream; nothing here computes on the CPU, and there is no fallback: a
missing library or a non-GPU tensor raises.

Entry points (same names as the C ABI):

* :func:`scan_block_step` -- one denoising step of the active block
  (Sec. 4, Eq. partial-reverse): forward branch continued from the cached state,
  block-local reverse branch from zero, summed.
* :func:`commit_boundary` -- block finalisation: the clean block's forward state
  replaces the cached one (Sec. 4, Eq. boundary-state).
* :func:`scan_full_window` -- the full-sequence bidirectional scan with no cache
  (the DiffuMamba-style contrast).
* :func:`prefill` -- summarise a long clean prefix into the cached states in one call.
* :func:`cache_reset` -- empty the given cache slots.

:class:`Cache` bundles a state pool with its host-side bookkeeping.
"""
from __future__ import annotations

import ctypes
import os
import re

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libbdlm.so")
BIND_PATH = os.path.join(_HERE, "_bind.so")
HEADER_PATH = os.path.join(os.path.dirname(_HERE), "include", "bdlm.h")

HEADDIM = 64
MAX_BLOCK_LEN = 64
MAX_SLOT_ROWS = 256
SCRATCH_BYTES = 64 << 20     # BDLM_SCRATCH_BYTES: the no-allocation prefill's device scratch
DTYPE_F32 = 0
DTYPE_BF16 = 1

OK, E_NULL, E_SHAPE, E_DTYPE, E_ALIGN, E_OFFSET, E_SLOT, E_LAUNCH, E_WORKSPACE = \
    0, -1, -2, -3, -4, -5, -6, -7, -8


class BdlmError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where}: {strerror(code)} (status {code})")


class Desc(ctypes.Structure):
    """Mirror of ``bdlm_desc_t``."""
    _fields_ = [
        ("batch", ctypes.c_int64),
        ("nheads", ctypes.c_int64),
        ("headdim", ctypes.c_int64),
        ("dstate", ctypes.c_int64),
        ("ngroups", ctypes.c_int64),
        ("block_len", ctypes.c_int64),
        ("in_dtype", ctypes.c_int32),
        ("reserved", ctypes.c_int32),
        ("x_stride", ctypes.c_int64 * 3),
        ("dt_stride", ctypes.c_int64 * 2),
        ("bc_stride", ctypes.c_int64 * 3),
    ]


_lib = None


def lib() -> ctypes.CDLL:
    """The loaded libbdlm.so (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with "
                               "`python -m paper_2607_02805_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        vp, fp = ctypes.c_void_p, ctypes.c_void_p
        i64, i32p = ctypes.c_int64, ctypes.POINTER(ctypes.c_int32)
        i64p = ctypes.POINTER(ctypes.c_int64)
        dp = ctypes.POINTER(Desc)
        L.bdlm_abi_version.restype = ctypes.c_int
        L.bdlm_strerror.argtypes = [ctypes.c_int]
        L.bdlm_strerror.restype = ctypes.c_char_p
        L.bdlm_desc_init.argtypes = [dp, i64, i64, i64, i64, i64, i64, ctypes.c_int32]
        L.bdlm_check_block_step.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, i64, i32p, fp]
        L.bdlm_check_commit.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, i64, i32p, i64p, i64p,
                                        i64]
        L.bdlm_scan_block_step.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, i64, i32p, fp, vp]
        L.bdlm_commit_boundary.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, i64, i32p, i64p,
                                           i64p, i64, fp, vp]
        L.bdlm_cache_reset.argtypes = [fp, i64, i64, i32p, i64, i64p, i64p, vp]
        L.bdlm_state_pack.argtypes = [fp, fp, i64, i64, vp]
        L.bdlm_state_unpack.argtypes = [fp, fp, i64, i64, vp]
        L.bdlm_conv_workspace.argtypes = [dp, i64p]
        L.bdlm_check_conv_block_step.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, fp, fp, fp, i64,
                                                 i32p, fp, vp, i64]
        L.bdlm_conv_block_step.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, fp, fp, fp, i64, i32p,
                                           fp, vp, i64, vp]
        L.bdlm_check_conv_commit.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, fp, fp, fp, i64, i32p,
                                             i64p, i64p, i64, fp, vp, i64]
        L.bdlm_conv_commit_boundary.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, fp, fp, fp, i64,
                                                i32p, i64p, i64p, i64, fp, vp, i64, vp]
        L.bdlm_check_block_step_sep.argtypes = [dp, vp, vp, fp, vp, vp, fp, vp, vp, fp, vp, vp,
                                                fp, fp, i64, i32p, fp]
        L.bdlm_scan_block_step_sep.argtypes = [dp, vp, vp, fp, vp, vp, fp, vp, vp, fp, vp, vp, fp,
                                               fp, i64, i32p, fp, vp]
        L.bdlm_boundary_states_workspace.argtypes = [dp, i64, i64p]
        L.bdlm_check_block_boundary_states.argtypes = [dp, i64, vp, vp, fp, vp, vp, fp, fp, fp,
                                                       fp, vp, i64]
        L.bdlm_block_boundary_states.argtypes = [dp, i64, vp, vp, fp, vp, vp, fp, fp, fp, fp, vp,
                                                 i64, vp]
        L.bdlm_full_window_workspace.argtypes = [dp, i64p]
        L.bdlm_prefill_workspace.argtypes = [dp, i64p]
        L.bdlm_check_full_window.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, vp, i64]
        L.bdlm_scan_full_window.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, fp, vp, i64, vp]
        L.bdlm_check_prefill.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, i64, i32p, i64p, i64p,
                                         i64, i64, fp, vp, i64]
        L.bdlm_prefill.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, i64, i32p, i64p, i64p, i64,
                                   i64, fp, vp, i64, vp]
        L.bdlm_commit_step.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, vp, vp, vp, vp, fp, i64,
                                       i32p, i64p, i64p, i64, fp, fp, vp]
        L.bdlm_check_commit_step.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, vp, vp, vp, vp, fp,
                                             i64, i32p, i64p, i64p, i64, fp, fp]
        L.bdlm_prefill_noalloc.argtypes = [dp, vp, vp, fp, vp, vp, fp, fp, i64, i32p, i64p, i64p,
                                           i64, i64, fp, vp]
        f32 = ctypes.c_float
        L.bdlm_check_gated_rmsnorm.argtypes = [i64, i64, i64, i64, ctypes.c_int32, fp, vp, i64,
                                               i64, fp, f32, fp]
        L.bdlm_gated_rmsnorm.argtypes = [i64, i64, i64, i64, ctypes.c_int32, fp, vp, i64, i64, fp,
                                         f32, fp, vp]
        for name in ("bdlm_desc_init", "bdlm_check_block_step", "bdlm_check_commit",
                     "bdlm_check_gated_rmsnorm", "bdlm_gated_rmsnorm",
                     "bdlm_scan_block_step", "bdlm_commit_boundary", "bdlm_cache_reset",
                     "bdlm_state_pack", "bdlm_state_unpack", "bdlm_check_full_window",
                     "bdlm_scan_full_window", "bdlm_check_prefill", "bdlm_prefill",
                     "bdlm_full_window_workspace", "bdlm_prefill_workspace",
                     "bdlm_boundary_states_workspace", "bdlm_check_block_boundary_states",
                     "bdlm_block_boundary_states", "bdlm_check_block_step_sep",
                     "bdlm_scan_block_step_sep", "bdlm_conv_workspace",
                     "bdlm_check_conv_block_step", "bdlm_conv_block_step",
                     "bdlm_check_conv_commit", "bdlm_conv_commit_boundary",
                     "bdlm_prefill_noalloc", "bdlm_commit_step", "bdlm_check_commit_step"):
            getattr(L, name).restype = ctypes.c_int
        if L.bdlm_abi_version() != 1:
            raise RuntimeError("libbdlm ABI version mismatch")
        _lib = L
    return _lib


_marshal = None


def _native():
    """The native marshalling (csrc/bdlm_bind.cpp): functions named as those here, which take
    the plain case of a call and answer NotImplemented to every other."""
    global _marshal
    if _marshal is None:
        lib()
        _torch()
        if not os.path.exists(BIND_PATH):
            raise RuntimeError(f"{BIND_PATH} is missing: build it with "
                               "`python -m paper_2607_02805_amd.build`")
        from . import _bind
        _marshal = _bind
    return _marshal


def _answer(got, where: str):
    """The result of a native call that was not NotImplemented: an int is a failure's status."""
    if type(got) is int:
        raise BdlmError(got, where)
    return got


def strerror(code: int) -> str:
    return lib().bdlm_strerror(int(code)).decode()


def header_functions() -> list[str]:
    """Names of the functions ``include/bdlm.h`` declares."""
    text = open(HEADER_PATH).read()
    return sorted(set(re.findall(r"^\s*(?:const\s+)?\w+\s*\*?\s*(bdlm_\w+)\s*\(", text, re.M)))


# ------------------------------------------------------------------ marshalling
def _torch():
    import torch
    return torch


def _dev_ptr(t, what: str) -> int:
    if not t.is_cuda:
        raise ValueError(f"{what} must be a GPU tensor (no CPU path exists)")
    return t.data_ptr()


def _stream_handle(stream) -> int | None:
    torch = _torch()
    s = torch.cuda.current_stream() if stream is None else stream
    return s.cuda_stream


def _desc(x, dt, Bm, Cm) -> Desc:
    torch = _torch()
    if x.dim() != 4 or dt.dim() != 3 or Bm.dim() != 4 or Cm.dim() != 4:
        raise ValueError("x [B,L,H,P], dt [B,L,H], B and C [B,L,G,N] expected")
    if not (x.dtype == dt.dtype == Bm.dtype == Cm.dtype):
        raise ValueError("x, dt, B and C must share one dtype")
    if x.dtype == torch.bfloat16:
        dty = DTYPE_BF16
    elif x.dtype == torch.float32:
        dty = DTYPE_F32
    else:
        raise ValueError(f"activations must be bfloat16 or float32, got {x.dtype}")
    bsz, L, H, P = x.shape
    G, N = Bm.shape[2], Bm.shape[3]
    if tuple(dt.shape) != (bsz, L, H) or tuple(Bm.shape) != (bsz, L, G, N) \
            or tuple(Cm.shape) != tuple(Bm.shape):
        raise ValueError("inconsistent activation shapes")
    d = Desc()
    if bsz * L == 0:
        # nothing is read: the strides of an empty tensor carry no meaning
        lib().bdlm_desc_init(ctypes.byref(d), bsz, H, P, N, G, L, dty)
        return d
    if x.stride(3) != 1 or dt.stride(2) != 1 or Bm.stride(3) != 1:
        raise ValueError("innermost dimension of x, dt, B must be unit stride")
    if tuple(Cm.stride()) != tuple(Bm.stride()):
        raise ValueError("B and C must share strides")
    d.batch, d.nheads, d.headdim, d.dstate, d.ngroups, d.block_len = bsz, H, P, N, G, L
    d.in_dtype, d.reserved = dty, 0
    d.x_stride[:] = list(x.stride()[:3])
    d.dt_stride[:] = list(dt.stride()[:2])
    d.bc_stride[:] = list(Bm.stride()[:3])
    return d


def _f32_vec(t, H, what):
    torch = _torch()
    if t.dtype != torch.float32 or t.dim() != 1 or t.shape[0] != H or not t.is_contiguous():
        raise ValueError(f"{what} must be a contiguous float32 [{H}] tensor")
    return _dev_ptr(t, what)


def pool_shape(nslots: int, nheads: int, dstate: int) -> tuple:
    """Shape of a state pool tensor: [nslots, nheads, dstate/4, 64, 4] (the pool layout of
    include/bdlm.h: state element s[p][n] at [.., n // 4, p, n % 4])."""
    return (nslots, nheads, dstate // 4, HEADDIM, 4)


def _pool(h_pool, H, N):
    torch = _torch()
    if h_pool.dtype != torch.float32 or not h_pool.is_contiguous() or h_pool.dim() != 5 \
            or tuple(h_pool.shape[1:]) != pool_shape(1, H, N)[1:]:
        raise ValueError(f"h_pool must be a contiguous float32 {pool_shape('nslots', H, N)} "
                         "tensor")
    return _dev_ptr(h_pool, "h_pool")


def _slots(slot_idx, rows: int):
    """Host int32 copy of ``slot_idx`` (one cache slot per batch row) and its pointer.
    The C ABI reads exactly ``rows`` entries, so any other length is refused here."""
    if slot_idx is None:
        return None, None
    arr = np.ascontiguousarray(np.asarray(slot_idx, dtype=np.int32))
    if arr.ndim != 1 or arr.shape[0] != rows:
        raise ValueError(f"slot_idx must be a 1-D sequence of exactly {rows} slot indices, "
                         f"got shape {arr.shape}")
    return arr, arr.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))


def _out(t, shape: tuple, what: str, device=None):
    """A float32 output: allocated when ``t`` is None or True, else checked to be a
    contiguous float32 tensor of exactly ``shape`` (the kernels write every element of
    that shape; a smaller buffer would be written past its end)."""
    torch = _torch()
    if t is None or t is True:
        return torch.empty(shape, dtype=torch.float32, device=device)
    if not torch.is_tensor(t) or t.dtype != torch.float32 or not t.is_contiguous() \
            or tuple(t.shape) != tuple(shape):
        got = (tuple(t.shape), t.dtype, t.is_contiguous()) if torch.is_tensor(t) else type(t)
        raise ValueError(f"{what} must be a contiguous float32 tensor of shape {tuple(shape)}, "
                         f"got {got}")
    return t


def scan_block_step(x, dt, A, B, C, D, D_rev, h_pool, y=None, slot_idx=None, stream=None):
    """One active-block denoising step on the GPU; returns ``y`` (float32 [B, L, H, 64]).

    ``h_pool`` is read only; ``slot_idx`` (host ints, optional) maps batch rows to
    cache slots.  Work is enqueued on ``stream`` (default: torch's current stream).
    """
    got = _native().scan_block_step(x, dt, A, B, C, D, D_rev, h_pool, y, slot_idx, stream)
    if got is not NotImplemented:
        return _answer(got, "bdlm_scan_block_step")
    torch = _torch()
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    y = _out(y, (d.batch, d.block_len, H, HEADDIM), "y", x.device)
    keep, sp = _slots(slot_idx, d.batch)
    rc = lib().bdlm_scan_block_step(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _f32_vec(D_rev, H, "D_rev"),
        _pool(h_pool, H, N), h_pool.shape[0], sp, _dev_ptr(y, "y"), _stream_handle(stream))
    del keep
    if rc != OK:
        raise BdlmError(rc, "bdlm_scan_block_step")
    return y


def scan_block_step_sep(fwd, rev, h_pool, y=None, slot_idx=None, stream=None):
    """A denoising step whose reverse branch has its own inputs: ``fwd`` and ``rev`` are
    (x, dt, A, B, C, skip) tuples of the same shapes and strides; the forward branch
    continues the cached state with skip ``fwd[5]`` (D), the reverse branch runs inside
    the block from zero with skip ``rev[5]`` (D_rev).  Returns y (float32 [B, L, H, 64])."""
    x, dt, A, B, C, D = fwd
    xr, dtr, Ar, Br, Cr, Dr = rev
    got = _native().scan_block_step_sep(x, dt, A, B, C, D, xr, dtr, Ar, Br, Cr, Dr, h_pool, y,
                                        slot_idx, stream)
    if got is not NotImplemented:
        return _answer(got, "bdlm_scan_block_step_sep")
    torch = _torch()
    for a, b, what in ((x, xr, "x"), (dt, dtr, "dt"), (A, Ar, "A"), (B, Br, "B"), (C, Cr, "C"),
                       (D, Dr, "D")):
        if tuple(a.shape) != tuple(b.shape) or a.dtype != b.dtype:
            raise ValueError(f"forward and reverse {what} must have the same shape and dtype, got "
                             f"{tuple(a.shape)} {a.dtype} and {tuple(b.shape)} {b.dtype}")
    d = _desc(x, dt, B, C)
    dr = _desc(xr, dtr, Br, Cr)
    if (list(d.x_stride), list(d.dt_stride), list(d.bc_stride), d.in_dtype) != \
            (list(dr.x_stride), list(dr.dt_stride), list(dr.bc_stride), dr.in_dtype):
        raise ValueError("forward and reverse inputs must share shapes, strides and dtype")
    H, N = d.nheads, d.dstate
    y = _out(y, (d.batch, d.block_len, H, HEADDIM), "y", x.device)
    keep, sp = _slots(slot_idx, d.batch)
    rc = lib().bdlm_scan_block_step_sep(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _dev_ptr(xr, "x_rev"),
        _dev_ptr(dtr, "dt_rev"), _f32_vec(Ar, H, "A_rev"), _dev_ptr(Br, "B_rev"),
        _dev_ptr(Cr, "C_rev"), _f32_vec(Dr, H, "D_rev"), _pool(h_pool, H, N), h_pool.shape[0],
        sp, _dev_ptr(y, "y"), _stream_handle(stream))
    del keep
    if rc != OK:
        raise BdlmError(rc, "bdlm_scan_block_step_sep")
    return y


def conv_channels(nheads, ngroups, dstate) -> int:
    """Channels of the mixer's convolution: x (nheads * 64), then B and C (ngroups * dstate)."""
    return nheads * HEADDIM + 2 * ngroups * dstate


def _conv_args(d, conv_w, conv_b, conv_pool, workspace, device):
    torch = _torch()
    ch = conv_channels(d.nheads, d.ngroups, d.dstate)
    if conv_w.dtype != torch.float32 or tuple(conv_w.shape) != (ch, 4) or not conv_w.is_contiguous():
        raise ValueError(f"conv_w must be a contiguous float32 [{ch}, 4] tensor")
    if conv_b.dtype != torch.float32 or tuple(conv_b.shape) != (ch,) or not conv_b.is_contiguous():
        raise ValueError(f"conv_b must be a contiguous float32 [{ch}] tensor")
    if conv_pool.dtype != torch.float32 or conv_pool.dim() != 3 or \
            tuple(conv_pool.shape[1:]) != (3, ch) or not conv_pool.is_contiguous():
        raise ValueError(f"conv_pool must be a contiguous float32 [nslots, 3, {ch}] tensor")
    wp, wb, keep = _workspace(lib().bdlm_conv_workspace, d, workspace, device)
    return wp, wb, keep


def conv_block_step(x, dt, A, B, C, D, D_rev, conv_w, conv_b, conv_pool, h_pool, y=None,
                    slot_idx=None, stream=None, workspace=None):
    """A denoising step with the mixer's convolution: x, B, C are pre-convolution inputs;
    the forward branch's convolution continues from ``conv_pool`` (read only), the
    reverse branch's is zero-padded inside the block.  Returns y (float32 [B, L, H, 64])."""
    got = _native().conv_block_step(x, dt, A, B, C, D, D_rev, conv_w, conv_b, conv_pool,
                                    h_pool, y, slot_idx, stream, workspace)
    if got is not NotImplemented:
        return _answer(got, "bdlm_conv_block_step")
    torch = _torch()
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    y = _out(y, (d.batch, d.block_len, H, HEADDIM), "y", x.device)
    if conv_pool.shape[0] != h_pool.shape[0]:
        raise ValueError("conv_pool and h_pool must have the same slots")
    wp, wb, wkeep = _conv_args(d, conv_w, conv_b, conv_pool, workspace, x.device)
    keep, sp = _slots(slot_idx, d.batch)
    rc = lib().bdlm_conv_block_step(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _f32_vec(D_rev, H, "D_rev"),
        _dev_ptr(conv_w, "conv_w"), _dev_ptr(conv_b, "conv_b"), _dev_ptr(conv_pool, "conv_pool"),
        _pool(h_pool, H, N), h_pool.shape[0], sp, _dev_ptr(y, "y"), wp, wb, _stream_handle(stream))
    del keep, wkeep
    if rc != OK:
        raise BdlmError(rc, "bdlm_conv_block_step")
    return y


def conv_commit_boundary(x, dt, A, B, C, D, D_rev, conv_w, conv_b, conv_pool, h_pool, n_committed,
                         n_blocks, expected_block_index=-1, slot_idx=None, y_clean=None,
                         stream=None, workspace=None):
    """Commit with the mixer's convolution: the SSM states advance over the forward
    branch's convolved block and ``conv_pool`` keeps the last three pre-convolution rows."""
    got = _native().conv_commit_boundary(x, dt, A, B, C, D, D_rev, conv_w, conv_b, conv_pool,
                                         h_pool, n_committed, n_blocks, expected_block_index,
                                         slot_idx, y_clean, stream, workspace)
    if got is not NotImplemented:
        return _answer(got, "bdlm_conv_commit_boundary")
    torch = _torch()
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    nslots = h_pool.shape[0]
    if conv_pool.shape[0] != nslots:
        raise ValueError("conv_pool and h_pool must have the same slots")
    for a in (n_committed, n_blocks):
        if not isinstance(a, np.ndarray) or a.dtype != np.int64 or a.shape != (nslots,):
            raise ValueError(f"n_committed / n_blocks must be numpy int64 [{nslots}]")
    if y_clean is not None:
        y_clean = _out(y_clean, (d.batch, d.block_len, H, HEADDIM), "y_clean", x.device)
    wp, wb, wkeep = _conv_args(d, conv_w, conv_b, conv_pool, workspace, x.device)
    keep, sp = _slots(slot_idx, d.batch)
    i64p = ctypes.POINTER(ctypes.c_int64)
    rc = lib().bdlm_conv_commit_boundary(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _f32_vec(D_rev, H, "D_rev"),
        _dev_ptr(conv_w, "conv_w"), _dev_ptr(conv_b, "conv_b"), _dev_ptr(conv_pool, "conv_pool"),
        _pool(h_pool, H, N), nslots, sp, n_committed.ctypes.data_as(i64p),
        n_blocks.ctypes.data_as(i64p), int(expected_block_index),
        None if y_clean is None else _dev_ptr(y_clean, "y_clean"), wp, wb, _stream_handle(stream))
    del keep, wkeep
    if rc != OK:
        raise BdlmError(rc, "bdlm_conv_commit_boundary")
    return y_clean


def commit_boundary(x, dt, A, B, C, D, D_rev, h_pool, n_committed, n_blocks,
                    expected_block_index=-1, slot_idx=None, y_clean=None, stream=None):
    """Commit the clean block: ``h_pool`` updated in place, host bookkeeping advanced.

    ``n_committed`` / ``n_blocks`` are host numpy int64 [nslots] arrays, updated in
    place.  ``y_clean``: None (skip), True (allocate and return) or a float32 tensor.
    Returns ``y_clean`` (or None).
    """
    got = _native().commit_boundary(x, dt, A, B, C, D, D_rev, h_pool, n_committed, n_blocks,
                                    expected_block_index, slot_idx, y_clean, stream)
    if got is not NotImplemented:
        return _answer(got, "bdlm_commit_boundary")
    torch = _torch()
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    nslots = h_pool.shape[0]
    for a in (n_committed, n_blocks):
        if not isinstance(a, np.ndarray) or a.dtype != np.int64 or not a.flags.c_contiguous \
                or a.shape != (nslots,):
            raise ValueError(f"n_committed / n_blocks must be contiguous numpy int64 [{nslots}]")
    yp = None
    if y_clean is not None:
        y_clean = _out(y_clean, (d.batch, d.block_len, H, HEADDIM), "y_clean", x.device)
        yp = _dev_ptr(y_clean, "y_clean")
    keep, sp = _slots(slot_idx, d.batch)
    i64p = ctypes.POINTER(ctypes.c_int64)
    rc = lib().bdlm_commit_boundary(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _f32_vec(D_rev, H, "D_rev"),
        _pool(h_pool, H, N), nslots, sp, n_committed.ctypes.data_as(i64p),
        n_blocks.ctypes.data_as(i64p), int(expected_block_index), yp, _stream_handle(stream))
    del keep
    if rc != OK:
        raise BdlmError(rc, "bdlm_commit_boundary")
    return y_clean


def commit_step(clean, nxt, A, D, D_rev, h_pool, n_committed, n_blocks, expected_block_index=-1,
                slot_idx=None, y_clean=None, y_next=None, stream=None):
    """Commit the clean block, then run the next block's first denoising step from the
    committed state, in one call (``clean`` and ``nxt`` are (x, dt, B, C) tuples of the same
    shapes and strides).  Same results as :func:`commit_boundary` followed by
    :func:`scan_block_step`; for bf16 blocks of at most 32 tokens one launch reads each
    state once.  Returns (y_next, y_clean)."""
    x, dt, B, C = clean
    xn, dtn, Bn, Cn = nxt
    got = _native().commit_step(x, dt, B, C, xn, dtn, Bn, Cn, A, D, D_rev, h_pool, n_committed,
                                n_blocks, expected_block_index, slot_idx, y_clean, y_next, stream)
    if got is not NotImplemented:
        return _answer(got, "bdlm_commit_step")
    for a, b, what in ((x, xn, "x"), (dt, dtn, "dt"), (B, Bn, "B"), (C, Cn, "C")):
        if tuple(a.shape) != tuple(b.shape) or a.dtype != b.dtype or a.stride() != b.stride():
            raise ValueError(f"clean and next {what} must share shape, dtype and strides")
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    nslots = h_pool.shape[0]
    for a in (n_committed, n_blocks):
        if not isinstance(a, np.ndarray) or a.dtype != np.int64 or not a.flags.c_contiguous \
                or a.shape != (nslots,):
            raise ValueError(f"n_committed / n_blocks must be contiguous numpy int64 [{nslots}]")
    shape = (d.batch, d.block_len, H, HEADDIM)
    y_next = _out(y_next, shape, "y_next", x.device)
    if y_clean is not None:
        y_clean = _out(y_clean, shape, "y_clean", x.device)
    keep, sp = _slots(slot_idx, d.batch)
    i64p = ctypes.POINTER(ctypes.c_int64)
    rc = lib().bdlm_commit_step(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _f32_vec(D_rev, H, "D_rev"),
        _dev_ptr(xn, "x_next"), _dev_ptr(dtn, "dt_next"), _dev_ptr(Bn, "B_next"),
        _dev_ptr(Cn, "C_next"), _pool(h_pool, H, N), nslots, sp,
        n_committed.ctypes.data_as(i64p), n_blocks.ctypes.data_as(i64p),
        int(expected_block_index), None if y_clean is None else _dev_ptr(y_clean, "y_clean"),
        _dev_ptr(y_next, "y_next"), _stream_handle(stream))
    del keep
    if rc != OK:
        raise BdlmError(rc, "bdlm_commit_step")
    return y_next, y_clean


def _workspace_bytes(fn, d) -> int:
    n = ctypes.c_int64(0)
    rc = fn(ctypes.byref(d), ctypes.byref(n))
    if rc != OK:
        raise BdlmError(rc, fn.__name__)
    return int(n.value)


def _workspace(fn, d, workspace, device):
    """(pointer, bytes, keep-alive) of the sequence workspace: the caller's tensor, or a
    fresh one from torch's allocator when none is given."""
    torch = _torch()
    need = _workspace_bytes(fn, d)
    if workspace is None:
        if need == 0:
            return None, 0, None
        workspace = torch.empty(need, dtype=torch.uint8, device=device)
    if not workspace.is_contiguous():
        raise ValueError("workspace must be a contiguous tensor")
    return workspace.data_ptr(), workspace.numel() * workspace.element_size(), workspace


def full_window_workspace_bytes(batch, nheads, dstate, window) -> int:
    d = Desc()
    lib().bdlm_desc_init(ctypes.byref(d), batch, nheads, HEADDIM, dstate, 1, window, DTYPE_BF16)
    return _workspace_bytes(lib().bdlm_full_window_workspace, d)


def prefill_workspace_bytes(batch, nheads, dstate, length) -> int:
    d = Desc()
    lib().bdlm_desc_init(ctypes.byref(d), batch, nheads, HEADDIM, dstate, 1, length, DTYPE_BF16)
    return _workspace_bytes(lib().bdlm_prefill_workspace, d)


def scan_full_window(x, dt, A, B, C, D, D_rev, y=None, stream=None, workspace=None):
    """Full-window bidirectional scan with no cache: forward over the whole window from
    zero plus reverse over the whole window from zero.  x is [B, W, H, 64]; returns y
    (float32 [B, W, H, 64]).  ``workspace``: a device tensor of at least
    :func:`full_window_workspace_bytes` bytes, 256-byte aligned (default: allocated)."""
    got = _native().scan_full_window(x, dt, A, B, C, D, D_rev, y, stream, workspace)
    if got is not NotImplemented:
        return _answer(got, "bdlm_scan_full_window")
    torch = _torch()
    d = _desc(x, dt, B, C)
    H = d.nheads
    y = _out(y, (d.batch, d.block_len, H, HEADDIM), "y", x.device)
    L = lib()
    wp, wb, keep = _workspace(L.bdlm_full_window_workspace, d, workspace, x.device)
    rc = L.bdlm_scan_full_window(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _f32_vec(D_rev, H, "D_rev"),
        _dev_ptr(y, "y"), wp, wb, _stream_handle(stream))
    del keep
    if rc != OK:
        raise BdlmError(rc, "bdlm_scan_full_window")
    return y


def prefill(x, dt, A, B, C, D, h_pool, n_committed, n_blocks, expected_block_index=-1,
            blocks_in_prefix=0, slot_idx=None, y_fwd=None, stream=None, workspace=None):
    """Summarise a clean prefix x [B, T, H, 64] (any T) into the cached states, in place.
    Bookkeeping advances by T tokens and ``blocks_in_prefix`` blocks.  ``y_fwd``: None,
    True (allocate and return) or a float32 tensor for the forward outputs.
    ``workspace``: as for :func:`scan_full_window` (:func:`prefill_workspace_bytes`)."""
    got = _native().prefill(x, dt, A, B, C, D, h_pool, n_committed, n_blocks,
                            expected_block_index, blocks_in_prefix, slot_idx, y_fwd, stream,
                            workspace)
    if got is not NotImplemented:
        return _answer(got, "bdlm_prefill")
    torch = _torch()
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    nslots = h_pool.shape[0]
    for a in (n_committed, n_blocks):
        if not isinstance(a, np.ndarray) or a.dtype != np.int64 or not a.flags.c_contiguous \
                or a.shape != (nslots,):
            raise ValueError(f"n_committed / n_blocks must be contiguous numpy int64 [{nslots}]")
    if y_fwd is not None:
        y_fwd = _out(y_fwd, (d.batch, d.block_len, H, HEADDIM), "y_fwd", x.device)
    yp = None if y_fwd is None else _dev_ptr(y_fwd, "y_fwd")
    keep, sp = _slots(slot_idx, d.batch)
    L = lib()
    wp, wb, wkeep = _workspace(L.bdlm_prefill_workspace, d, workspace, x.device)
    i64p = ctypes.POINTER(ctypes.c_int64)
    rc = L.bdlm_prefill(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _pool(h_pool, H, N), nslots,
        sp, n_committed.ctypes.data_as(i64p), n_blocks.ctypes.data_as(i64p),
        int(expected_block_index), int(blocks_in_prefix), yp, wp, wb, _stream_handle(stream))
    del keep, wkeep
    if rc != OK:
        raise BdlmError(rc, "bdlm_prefill")
    return y_fwd


def prefill_noalloc(x, dt, A, B, C, D, h_pool, n_committed, n_blocks, expected_block_index=-1,
                    blocks_in_prefix=0, slot_idx=None, y_fwd=None, stream=None):
    """:func:`prefill` through ``bdlm_prefill_noalloc``: no workspace and no allocation, by
    the library or here (``y_fwd`` is None or a caller tensor), so it can run inside a HIP
    graph capture or a loop that must not allocate.  The segment states use the device
    scratch the library owns (``SCRATCH_BYTES`` per device); calls that overlap on one
    device race."""
    got = _native().prefill_noalloc(x, dt, A, B, C, D, h_pool, n_committed, n_blocks,
                                    expected_block_index, blocks_in_prefix, slot_idx, y_fwd,
                                    stream)
    if got is not NotImplemented:
        return _answer(got, "bdlm_prefill_noalloc")
    d = _desc(x, dt, B, C)
    H, N = d.nheads, d.dstate
    nslots = h_pool.shape[0]
    for a in (n_committed, n_blocks):
        if not isinstance(a, np.ndarray) or a.dtype != np.int64 or not a.flags.c_contiguous \
                or a.shape != (nslots,):
            raise ValueError(f"n_committed / n_blocks must be contiguous numpy int64 [{nslots}]")
    if y_fwd is True:
        raise ValueError("prefill_noalloc allocates nothing: pass y_fwd as a tensor or None")
    if y_fwd is not None:
        y_fwd = _out(y_fwd, (d.batch, d.block_len, H, HEADDIM), "y_fwd")
    yp = None if y_fwd is None else _dev_ptr(y_fwd, "y_fwd")
    keep, sp = _slots(slot_idx, d.batch)
    i64p = ctypes.POINTER(ctypes.c_int64)
    rc = lib().bdlm_prefill_noalloc(
        ctypes.byref(d), _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"), _pool(h_pool, H, N), nslots,
        sp, n_committed.ctypes.data_as(i64p), n_blocks.ctypes.data_as(i64p),
        int(expected_block_index), int(blocks_in_prefix), yp, _stream_handle(stream))
    del keep
    if rc != OK:
        raise BdlmError(rc, "bdlm_prefill_noalloc")
    return y_fwd


def block_boundary_states(x, dt, A, B, C, D, block_len, s_init=None, s_out=None, y_fwd=None,
                          stream=None, workspace=None):
    """States entering every block of a clean sequence x [B, K * block_len, H, 64]:
    returns ``s_out`` (float32, pool layout, [B * K, H, N/4, 64, 4]; state b * K + k is
    the forward state after blocks 0 .. k-1 of row b, k = 0 being ``s_init`` or zero)
    and, if ``y_fwd`` is True or a tensor, the forward outputs of the sequence."""
    torch = _torch()
    d = _desc(x, dt, B, C)
    T, H, N = d.block_len, d.nheads, d.dstate
    if block_len <= 0 or T % block_len != 0:
        raise ValueError("the sequence length must be a whole number of blocks")
    K = T // block_len
    d.block_len = block_len
    if s_out is None:
        s_out = torch.empty(pool_shape(d.batch * K, H, N), dtype=torch.float32, device=x.device)
    elif s_out.dtype != torch.float32 or not s_out.is_contiguous() \
            or s_out.numel() != d.batch * K * H * HEADDIM * N:
        raise ValueError(f"s_out must be a contiguous float32 tensor of {d.batch * K * H} states")
    if s_init is not None and (s_init.dtype != torch.float32 or not s_init.is_contiguous()
                               or s_init.numel() != d.batch * H * HEADDIM * N):
        raise ValueError(f"s_init must be a contiguous float32 tensor of {d.batch * H} states")
    if y_fwd is not None:
        y_fwd = _out(y_fwd, (d.batch, T, H, HEADDIM), "y_fwd", x.device)
    L = lib()
    need = ctypes.c_int64(0)
    rc = L.bdlm_boundary_states_workspace(ctypes.byref(d), K, ctypes.byref(need))
    if rc != OK:
        raise BdlmError(rc, "bdlm_boundary_states_workspace")
    if workspace is None and need.value > 0:
        workspace = torch.empty(need.value, dtype=torch.uint8, device=x.device)
    wp = None if workspace is None else workspace.data_ptr()
    wb = 0 if workspace is None else workspace.numel() * workspace.element_size()
    rc = L.bdlm_block_boundary_states(
        ctypes.byref(d), K, _dev_ptr(x, "x"), _dev_ptr(dt, "dt"), _f32_vec(A, H, "A"),
        _dev_ptr(B, "B"), _dev_ptr(C, "C"), _f32_vec(D, H, "D"),
        None if s_init is None else _dev_ptr(s_init, "s_init"), _dev_ptr(s_out, "s_out"),
        None if y_fwd is None else _dev_ptr(y_fwd, "y_fwd"), wp, wb, _stream_handle(stream))
    if rc != OK:
        raise BdlmError(rc, "bdlm_block_boundary_states")
    return (s_out, y_fwd) if y_fwd is not None else s_out


def all_block_forward(clean, noised, A, D, D_rev, block_len, s_init=None, want_clean_y=False,
                      stream=None):
    """The all-block training forward of one Mamba layer: ``clean`` and ``noised`` are
    (x, dt, B, C) of the same window [B, K * block_len, ...]; every noised block k is
    stepped (forward from the clean prefix's state before block k, reverse inside the
    block) in one batched block step.  Returns (y_noised [B, K * block_len, H, 64],
    s_out[, y_clean_forward])."""
    xc, dtc, Bc, Cc = clean
    xn, dtn, Bn, Cn = noised
    bsz, T = xn.shape[0], xn.shape[1]
    K = T // block_len
    out = block_boundary_states(xc, dtc, A, Bc, Cc, D, block_len, s_init=s_init,
                                y_fwd=True if want_clean_y else None, stream=stream)
    s_out = out[0] if want_clean_y else out

    def blocks(t):   # [B, K * L, ...] -> [B * K, L, ...] (a view when contiguous)
        return t.reshape(bsz * K, block_len, *t.shape[2:])
    y = scan_block_step(blocks(xn), blocks(dtn), A, blocks(Bn), blocks(Cn), D, D_rev, s_out,
                        stream=stream)
    y = y.reshape(bsz, T, *y.shape[2:])
    return (y, s_out, out[1]) if want_clean_y else (y, s_out)


def gated_rmsnorm(y, z, norm_w, eps=1e-5, ngroups=1, out=None, stream=None):
    """Gated RMS normalisation of a scan output (the Mamba-2 mixer's output path):
    ``out = norm_w * g / sqrt(mean_group(g^2) + eps)``, ``g = y * silu(z)``, per token over
    the ``nheads * 64`` channels in ``ngroups`` groups of whole heads.

    ``y`` float32 [B, L, H, 64] (or [B, L, H * 64]), contiguous; ``z`` bfloat16 or float32
    [B, L, H * 64] with unit channel stride (a slice of a projection output is fine);
    ``norm_w`` float32 [H * 64].  ``out`` may be ``y`` (in place).  Returns ``out``.
    """
    got = _native().gated_rmsnorm(y, z, norm_w, eps, ngroups, out, stream)
    if got is not NotImplemented:
        return _answer(got, "bdlm_gated_rmsnorm")
    torch = _torch()
    if y.dtype != torch.float32 or not y.is_contiguous() or y.dim() not in (3, 4):
        raise ValueError("y must be a contiguous float32 [B, L, H, 64] or [B, L, H*64] tensor")
    bsz, L = y.shape[0], y.shape[1]
    nch = y.shape[2] * y.shape[3] if y.dim() == 4 else y.shape[2]
    if nch % HEADDIM:
        raise ValueError("channels must be whole heads of 64")
    H = nch // HEADDIM
    if z.dim() != 3 or tuple(z.shape) != (bsz, L, nch):
        raise ValueError(f"z must be [B, L, {nch}]")
    if z.dtype == torch.bfloat16:
        zdt = DTYPE_BF16
    elif z.dtype == torch.float32:
        zdt = DTYPE_F32
    else:
        raise ValueError(f"z must be bfloat16 or float32, got {z.dtype}")
    if bsz * L and z.stride(2) != 1:
        raise ValueError("z must have unit channel stride")
    if norm_w.dtype != torch.float32 or tuple(norm_w.shape) != (nch,) or not norm_w.is_contiguous():
        raise ValueError(f"norm_w must be a contiguous float32 [{nch}] tensor")
    if out is None:
        out = torch.empty_like(y)
    elif out.dtype != torch.float32 or tuple(out.shape) != tuple(y.shape) or not out.is_contiguous():
        raise ValueError("out must be a contiguous float32 tensor shaped like y")
    empty = bsz * L == 0
    rc = lib().bdlm_gated_rmsnorm(
        bsz, L, H, int(ngroups), zdt, None if empty else _dev_ptr(y, "y"),
        None if empty else _dev_ptr(z, "z"), z.stride(0) if not empty else 0,
        z.stride(1) if not empty else 0, _dev_ptr(norm_w, "norm_w"), float(eps),
        None if empty else _dev_ptr(out, "out"), _stream_handle(stream))
    if rc != OK:
        raise BdlmError(rc, "bdlm_gated_rmsnorm")
    return out


def cache_reset(h_pool, slots=None, n_committed=None, n_blocks=None, stream=None):
    """Zero the given slots of ``h_pool`` (all if None) and their bookkeeping."""
    torch = _torch()
    if h_pool.dtype != torch.float32 or not h_pool.is_contiguous():
        raise ValueError("h_pool must be a contiguous float32 tensor")
    nslots = h_pool.shape[0]
    elems = h_pool[0].numel() if nslots else 0
    keep, sp = (None, None) if slots is None else _slots(slots, len(slots))
    i64p = ctypes.POINTER(ctypes.c_int64)
    rc = lib().bdlm_cache_reset(
        _dev_ptr(h_pool, "h_pool"), nslots, elems, sp, 0 if keep is None else len(keep),
        None if n_committed is None else n_committed.ctypes.data_as(i64p),
        None if n_blocks is None else n_blocks.ctypes.data_as(i64p), _stream_handle(stream))
    if rc != OK:
        raise BdlmError(rc, "bdlm_cache_reset")


def state_pack(rowmajor, pool=None, stream=None):
    """Row-major states [..., 64, dstate] (float32, GPU) -> a pool tensor [..., dstate/4, 64, 4]."""
    torch = _torch()
    if rowmajor.dtype != torch.float32 or not rowmajor.is_contiguous() or rowmajor.dim() < 2 \
            or rowmajor.shape[-2] != HEADDIM:
        raise ValueError("states must be a contiguous float32 [..., 64, dstate] tensor")
    N = rowmajor.shape[-1]
    lead = tuple(rowmajor.shape[:-2])
    if pool is None:
        pool = torch.empty(lead + (N // 4, HEADDIM, 4), dtype=torch.float32,
                           device=rowmajor.device)
    n = rowmajor.numel() // (HEADDIM * N)
    rc = lib().bdlm_state_pack(_dev_ptr(rowmajor, "rowmajor"), _dev_ptr(pool, "pool"), n, N,
                               _stream_handle(stream))
    if rc != OK:
        raise BdlmError(rc, "bdlm_state_pack")
    return pool


def state_unpack(pool, rowmajor=None, stream=None):
    """A pool tensor [..., dstate/4, 64, 4] -> row-major states [..., 64, dstate]."""
    torch = _torch()
    if pool.dtype != torch.float32 or not pool.is_contiguous() or pool.dim() < 3 \
            or tuple(pool.shape[-2:]) != (HEADDIM, 4):
        raise ValueError("pool must be a contiguous float32 [..., dstate/4, 64, 4] tensor")
    N = pool.shape[-3] * 4
    lead = tuple(pool.shape[:-3])
    if rowmajor is None:
        rowmajor = torch.empty(lead + (HEADDIM, N), dtype=torch.float32, device=pool.device)
    n = pool.numel() // (HEADDIM * N)
    rc = lib().bdlm_state_unpack(_dev_ptr(pool, "pool"), _dev_ptr(rowmajor, "rowmajor"), n, N,
                                 _stream_handle(stream))
    if rc != OK:
        raise BdlmError(rc, "bdlm_state_unpack")
    return rowmajor


class Cache:
    """A pool of per-sequence forward boundary states for one Mamba layer.

    ``h`` is a float32 GPU tensor in the pool layout, [nslots, nheads, dstate/4, 64, 4];
    ``n_committed`` and ``n_blocks`` are host int64 arrays (tokens / blocks summarised
    per slot).  :meth:`states` returns the states as row-major [nslots, nheads, 64, dstate].
    """

    def __init__(self, nslots: int, nheads: int, dstate: int, device="cuda", ngroups: int = 0):
        """``ngroups`` > 0 also keeps the mixer's convolution rows (``conv``, float32
        [nslots, 3, channels]) for :meth:`conv_step` / :meth:`conv_commit`."""
        torch = _torch()
        self.h = torch.zeros(pool_shape(nslots, nheads, dstate), dtype=torch.float32,
                             device=device)
        self.conv = None
        if ngroups > 0:
            self.conv = torch.zeros((nslots, 3, conv_channels(nheads, ngroups, dstate)),
                                    dtype=torch.float32, device=device)
        self.n_committed = np.zeros(nslots, np.int64)
        self.n_blocks = np.zeros(nslots, np.int64)

    def conv_step(self, x, dt, A, B, C, D, D_rev, conv_w, conv_b, y=None, slot_idx=None,
                  stream=None):
        return conv_block_step(x, dt, A, B, C, D, D_rev, conv_w, conv_b, self.conv, self.h, y,
                               slot_idx, stream)

    def conv_commit(self, x, dt, A, B, C, D, D_rev, conv_w, conv_b, expected_block_index=-1,
                    slot_idx=None, y_clean=None, stream=None):
        return conv_commit_boundary(x, dt, A, B, C, D, D_rev, conv_w, conv_b, self.conv, self.h,
                                    self.n_committed, self.n_blocks, expected_block_index,
                                    slot_idx, y_clean, stream)

    def step(self, x, dt, A, B, C, D, D_rev, y=None, slot_idx=None, stream=None):
        return scan_block_step(x, dt, A, B, C, D, D_rev, self.h, y, slot_idx, stream)

    def commit(self, x, dt, A, B, C, D, D_rev, expected_block_index=-1, slot_idx=None,
               y_clean=None, stream=None):
        return commit_boundary(x, dt, A, B, C, D, D_rev, self.h, self.n_committed,
                               self.n_blocks, expected_block_index, slot_idx, y_clean, stream)

    def prefill(self, x, dt, A, B, C, D, expected_block_index=-1, blocks_in_prefix=0,
                slot_idx=None, y_fwd=None, stream=None, workspace=None):
        return prefill(x, dt, A, B, C, D, self.h, self.n_committed, self.n_blocks,
                       expected_block_index, blocks_in_prefix, slot_idx, y_fwd, stream,
                       workspace)

    def reset(self, slots=None, stream=None):
        cache_reset(self.h, slots, self.n_committed, self.n_blocks, stream)
        if self.conv is not None:
            cache_reset(self.conv, slots, stream=stream)

    def states(self, stream=None):
        """The cached states as a row-major [nslots, nheads, 64, dstate] tensor."""
        return state_unpack(self.h, stream=stream)

    def load_states(self, rowmajor, stream=None):
        """Overwrite the states from a row-major [nslots, nheads, 64, dstate] tensor."""
        state_pack(rowmajor.contiguous(), self.h, stream=stream)

    def state_dict(self) -> dict:
        """Checkpoint: the states (on the host) and the bookkeeping."""
        sd = {"h": self.h.detach().cpu(), "n_committed": self.n_committed.copy(),
              "n_blocks": self.n_blocks.copy()}
        if self.conv is not None:
            sd["conv"] = self.conv.detach().cpu()
        return sd

    def load_state_dict(self, sd: dict) -> None:
        if tuple(sd["h"].shape) != tuple(self.h.shape):
            raise ValueError("checkpoint shape does not match this cache")
        self.h.copy_(sd["h"])
        if self.conv is not None:
            self.conv.copy_(sd["conv"])
        self.n_committed[:] = sd["n_committed"]
        self.n_blocks[:] = sd["n_blocks"]
