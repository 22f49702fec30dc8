"""Thin binding over libsar_mi355x.so: same names as include/sar_mi355x.h.  The calls of a step go through _binding.so, which
checks their tensors and hands them over; handles are built, and the rarer calls made, over ctypes.

Argument marshalling only -- every step of the path runs in the library's HIP
kernels.  torch is used for device memory (``tensor.data_ptr()``) and for the
current stream.  If the shared library is missing the import of any function
here raises; there is no CPU fallback.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libsar_mi355x.so")

SAR_OK = 0
SAR_ERR_INVALID_ARG = -1
SAR_ERR_UNSUPPORTED = -2
SAR_ERR_HIP = -3
SAR_ERR_STATE = -4
SAR_F32 = 0
SAR_BF16 = 1
SAR_ACT_NONE = 0
SAR_ACT_RELU = 1
SAR_MAX_BLOCKS = 64      # blocks of an all-blocks call (handles built with SAR_BUILD_FUSED)
SAR_MAX_PARTS = 256      # partitions of any handle
SAR_BUILD_TRANSPOSE = 1
SAR_BUILD_FUSED = 2
SAR_BUILD_SKIP_UNTOUCHED = 4
SAR_BUILD_COMPACT = 8
SAR_BUILD_SINGLES = 16
SAR_BUILD_NO_SINGLES = 32

_c_i64 = ctypes.c_int64
_c_int = ctypes.c_int
_vp = ctypes.c_void_p


class SarError(RuntimeError):
    def __init__(self, code: int, text: str):
        super().__init__("sar error %d: %s" % (code, text))
        self.code = code


class BlockView(ctypes.Structure):
    _fields_ = [
        ("n_dst", _c_i64), ("n_src", _c_i64), ("nnz", _c_i64),
        ("indptr", _vp), ("indices", _vp), ("t_indptr", _vp), ("t_indices", _vp),
        ("rows", _vp), ("n_rows", _c_i64), ("n_long", _c_i64),
        ("t_rows", _vp), ("n_t_rows", _c_i64), ("n_t_long", _c_i64),
        ("touched", _vp), ("t_rank", _vp),
    ]


_lib = None


def lib() -> ctypes.CDLL:
    """The loaded library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                "%s is missing: build it with `python -m paper_2111_06483_amd.build` "
                "(there is no fallback path)" % LIB_PATH)
        loaded = ctypes.CDLL(LIB_PATH)
        for name, sig in _SIGNATURES.items():
            getattr(loaded, name).argtypes = [_CTYPES[c] for c in sig]   # fails early if a symbol is missing
        loaded.sar_last_error.restype = ctypes.c_char_p
        _lib = loaded
    return _lib


_native = None


def native():
    """The loaded binding of the hot calls; raises if it has not been built, or not for this interpreter and torch."""
    global _native
    if _native is None:
        lib()
        how = "build it with `python -m paper_2111_06483_amd.build` (there is no fallback path)"
        try:
            from . import _binding, build
        except ImportError as e:
            raise RuntimeError("_binding.so does not load (%s): %s" % (e, how)) from e
        built_for, here = getattr(_binding, "built_for", "another version"), build.binding_for()
        if built_for != here:
            raise RuntimeError("_binding.so reads tensors by the headers of %s, and this is %s: %s" % (built_for, here, how))
        _native = _binding
    return _native


# Parameter types of the entry points, declared once so that a call hands over plain Python values: p address,
# i int, l int64_t, z size_t, f float.
_SIGNATURES = {
    "sar_last_error": "", "sar_version": "",
    "sar_blocks_build": "ppilpliiipp", "sar_blocks_wrap": "ilpppipp", "sar_blocks_subset": "pplipp",
    "sar_blocks_info": "ppp", "sar_blocks_get": "pip", "sar_blocks_singles": "pppppp", "sar_blocks_degree": "pp",
    "sar_blocks_free": "p", "sar_release_memory": "",
    "sar_spmm_block": "pipiipp", "sar_spmm_end": "pippipilip", "sar_spmm_all": "ppiiipipp", "sar_act_bwd": "ppipilp",
    "sar_spmm_bwd_block": "pipiiipp", "sar_spmm_bwd_all": "ppiiipp", "sar_error_add": "ppipilip",
    "sar_gat_scores": "piliippp", "sar_gat_fwd_begin": "pppliip", "sar_gat_fwd_block": "pippppiiifpppp",
    "sar_gat_fwd_end": "pppippiliip", "sar_gat_fwd_all": "pppppiiifippp", "sar_gat_workspace_bytes": "lliip",
    "sar_gat_bwd_begin": "ppppipippliip", "sar_gat_bwd_block": "pipppppiiifpppppzp",
    "sar_gat_bwd_all": "ppppppiiifpppppzp", "sar_gat_bwd_end": "pppppppiliipzp",
    "sar_gat_bwd_end_noalloc": "pppppppiliip",
    "sar_linear_fwd": "pppiliiiippppp", "sar_linear_bwd": "pppppiliipzp", "sar_linear_bwd_rows": "ppplppiipppilippzp",
    "sar_linear_workspace_bytes": "liip",
}
_CTYPES = {"p": _vp, "i": _c_int, "l": _c_i64, "z": ctypes.c_size_t, "f": ctypes.c_float}
EXPORTS = list(_SIGNATURES)


def _same_shape(a: torch.Tensor, b: Optional[torch.Tensor]) -> None:
    """The C side takes one size for both: refuse a second tensor of another shape or dtype."""
    if b is not None and (a.shape != b.shape or a.dtype != b.dtype):
        raise SarError(SAR_ERR_INVALID_ARG, "tensors of shape %s %s and %s %s must match"
                       % (tuple(a.shape), a.dtype, tuple(b.shape), b.dtype))


def _check(rc: int) -> None:
    if rc != SAR_OK:
        raise SarError(rc, lib().sar_last_error().decode())


def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    if t is None:
        return None
    assert t.is_contiguous(), "tensors passed to the library must be contiguous"
    return t.data_ptr()


# The address of the current stream without the Stream object around it, which took a third of the host
# time of a short pass (2 of 12 us per call).
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream() -> Optional[int]:
    if _raw_stream is not None and torch.cuda.is_initialized():
        return _raw_stream(torch.cuda.current_device())
    if torch.cuda.is_available():
        return torch.cuda.current_stream().cuda_stream
    return None


def dtype_code(dt: torch.dtype) -> int:
    if dt == torch.float32:
        return SAR_F32
    if dt == torch.bfloat16:
        return SAR_BF16
    raise SarError(SAR_ERR_UNSUPPORTED, "dtype %s" % dt)


def _ptr_array(ts: Sequence[Optional[torch.Tensor]], what: str, dtype: torch.dtype):
    """Host array of device pointers, one per block.  The C side reinterprets the memory, so every
    entry must be what the call assumes: on the device, contiguous, of `dtype`."""
    ptrs = []
    for k, t in enumerate(ts):
        if t is None:
            ptrs.append(None)
            continue
        if not t.is_cuda or not t.is_contiguous():
            raise SarError(SAR_ERR_INVALID_ARG, "%s[%d] must be a contiguous device tensor" % (what, k))
        if t.dtype != dtype:
            raise SarError(SAR_ERR_INVALID_ARG, "%s[%d] is %s, the call needs %s" % (what, k, t.dtype, dtype))
        ptrs.append(t.data_ptr())
    return (_vp * len(ptrs))(*ptrs)


class Blocks:
    """Owner of a sar_blocks_t handle (freed on ``close`` / garbage collection)."""

    def __init__(self, handle: _vp, keep=(), flags: int = 0):
        self._h = handle
        self._addr = handle.value
        self._keep = keep   # tensors borrowed by a wrapped handle
        self.flags = flags
        self._n_src = {}
        self._n_err = {}
        P, n = _c_int(0), _c_i64(0)
        _check(lib().sar_blocks_info(self._h, ctypes.byref(P), ctypes.byref(n)))
        self.P, self.n_dst = P.value, n.value

    @property
    def handle(self) -> _vp:
        if self._h is None:
            raise SarError(SAR_ERR_STATE, "blocks handle already freed")
        return self._h

    def view(self, q: int) -> BlockView:
        v = BlockView()
        _check(lib().sar_blocks_get(self.handle, q, ctypes.byref(v)))
        return v

    def n_src(self, q: int) -> int:
        if q not in self._n_src:
            self._n_src[q] = int(self.view(q).n_src)
        return self._n_src[q]

    def check_rows(self, q: int, *tensors) -> None:
        """Host-side guard: per-source tensors of block q must have n_src rows."""
        n = self._n_src.get(q)
        if n is None:
            n = self.n_src(q)
        for t in tensors:
            if t is not None and t.size(0) != n:
                raise SarError(SAR_ERR_INVALID_ARG, "block %d has %d sources, tensor has %d rows"
                               % (q, n, t.size(0)))

    def n_err_rows(self, q: int) -> int:
        """Rows of block q's dZ_q / dt_q: n_src, or n_t_rows on a SAR_BUILD_COMPACT handle."""
        if not (self.flags & SAR_BUILD_COMPACT):
            return self.n_src(q)
        if q not in self._n_err:
            self._n_err[q] = int(self.view(q).n_t_rows)
        return self._n_err[q]

    def check_err_rows(self, q: int, *tensors) -> None:
        n = self._n_err.get(q)
        if n is None:
            n = self._n_err[q] = self.n_err_rows(q)
        for t in tensors:
            if t is not None and t.size(0) != n:
                raise SarError(SAR_ERR_INVALID_ARG, "block %d's error has %d rows, tensor has %d"
                               % (q, n, t.size(0)))

    def check_dst(self, *tensors) -> None:
        for t in tensors:
            if t is not None and t.size(0) != self.n_dst:
                raise SarError(SAR_ERR_INVALID_ARG, "handle has %d destinations, tensor has %d rows"
                               % (self.n_dst, t.size(0)))

    def close(self) -> None:
        if self._h is not None:
            lib().sar_blocks_free(self._h)
            self._h = self._addr = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def device_array(ptr: Optional[int], count: int, dtype=torch.int32, device="cuda") -> torch.Tensor:
    """Copy of `count` elements at device address `ptr` (for inspection in tests)."""
    out = torch.empty(count, dtype=dtype, device=device)
    if count:
        nbytes = count * out.element_size()
        rc = _hip().hipMemcpy(_vp(out.data_ptr()), _vp(ptr), ctypes.c_size_t(nbytes), _c_int(3))
        if rc != 0:
            raise RuntimeError("hipMemcpy failed: %d" % rc)
    return out


_hiprt = None


def _hip():
    global _hiprt
    if _hiprt is None:
        _hiprt = ctypes.CDLL("libamdhip64.so")
    return _hiprt


# ------------------------------------------------------------------ blocks

def sar_blocks_build(src: torch.Tensor, dst: torch.Tensor, part: torch.Tensor, P: int, p: int,
                     flags: int = SAR_BUILD_TRANSPOSE | SAR_BUILD_FUSED) -> Blocks:
    assert src.dtype == dst.dtype and src.dtype in (torch.int32, torch.int64)
    assert part.dtype == torch.int32
    h = _vp(None)
    _check(lib().sar_blocks_build(_ptr(src), _ptr(dst), src.element_size(), src.numel(),
                                  _ptr(part), part.numel(), P, p, flags,
                                  _stream(), ctypes.byref(h)))
    return Blocks(h, flags=flags)


def sar_blocks_wrap(n_dst: int, n_src: Sequence[int], indptr: Sequence[torch.Tensor],
                    indices: Sequence[torch.Tensor],
                    flags: int = SAR_BUILD_TRANSPOSE | SAR_BUILD_FUSED) -> Blocks:
    P = len(indptr)
    ns = (_c_i64 * P)(*[int(x) for x in n_src])
    h = _vp(None)
    _check(lib().sar_blocks_wrap(P, n_dst, ns, _ptr_array(indptr, "indptr", torch.int32),
                                 _ptr_array(indices, "indices", torch.int32), flags, _stream(),
                                 ctypes.byref(h)))
    return Blocks(h, keep=(list(indptr), list(indices)), flags=flags)


def sar_blocks_subset(b: Blocks, dst_ids: torch.Tensor,
                      flags: int = SAR_BUILD_TRANSPOSE | SAR_BUILD_FUSED) -> Blocks:
    if dst_ids.dtype != torch.int32 or dst_ids.dim() != 1 or not dst_ids.is_contiguous():
        raise SarError(SAR_ERR_INVALID_ARG, "dst_ids must be a contiguous 1-d int32 tensor")
    h = _vp(None)
    _check(lib().sar_blocks_subset(b.handle, _ptr(dst_ids), dst_ids.numel(), flags, _stream(),
                                   ctypes.byref(h)))
    return Blocks(h, flags=flags)


def sar_blocks_n_singles(b: Blocks) -> int:
    """Length of the handle's list of single-edge sources (0: not built)."""
    n = _c_i64(0)
    _check(lib().sar_blocks_singles(b.handle, ctypes.byref(n), None, None, None, None))
    return int(n.value)


def sar_blocks_singles(b: Blocks):
    """(dst, src, row, tag_shift) of the handle's destination-major list of the sources that have one
    edge in their block (copies, for inspection); three empty tensors where the list was not built."""
    n, ts = _c_i64(0), _c_int(0)
    pd, ps, pr = _vp(None), _vp(None), _vp(None)
    _check(lib().sar_blocks_singles(b.handle, ctypes.byref(n), ctypes.byref(pd), ctypes.byref(ps), ctypes.byref(pr),
                                    ctypes.byref(ts)))
    return (device_array(pd.value, n.value), device_array(ps.value, n.value), device_array(pr.value, n.value),
            ts.value)


def sar_blocks_degree(b: Blocks) -> torch.Tensor:
    p = _vp(None)
    _check(lib().sar_blocks_degree(b.handle, ctypes.byref(p)))
    return device_array(p.value, b.n_dst)


def sar_release_memory() -> None:
    """Free the device memory the library keeps for coming builder calls."""
    _check(lib().sar_release_memory())


# -------------------------------------------------------------------- spmm

def sar_spmm_block(b: Blocks, q: int, Zq: torch.Tensor, acc: torch.Tensor) -> None:
    b.check_rows(q, Zq)
    b.check_dst(acc)
    _check(lib().sar_spmm_block(b.handle, q, _ptr(Zq), dtype_code(Zq.dtype),
                                Zq.shape[-1], _ptr(acc), _stream()))


def sar_spmm_end(deg: torch.Tensor, mean: bool, acc: torch.Tensor, out: torch.Tensor,
                 residual: Optional[torch.Tensor] = None, act: int = SAR_ACT_NONE) -> None:
    _same_shape(out, residual)
    _check(lib().sar_spmm_end(_ptr(deg), int(mean), _ptr(acc), _ptr(residual), act, _ptr(out),
                              dtype_code(out.dtype), acc.shape[0], acc.shape[1],
                              _stream()))


def sar_spmm_all(b: Blocks, Zq: Sequence[torch.Tensor], mean: bool, out: torch.Tensor,
                 residual: Optional[torch.Tensor] = None, act: int = SAR_ACT_NONE) -> None:
    native().spmm_all(b, Zq, mean, out, residual, act)


def sar_act_bwd(h: torch.Tensor, dH: torch.Tensor, act: int, G: torch.Tensor) -> None:
    native().act_bwd(h, dH, act, G)


def sar_spmm_bwd_block(b: Blocks, q: int, G: torch.Tensor, mean: bool, dZq: torch.Tensor) -> None:
    b.check_err_rows(q, dZq)
    b.check_dst(G)
    _check(lib().sar_spmm_bwd_block(b.handle, q, _ptr(G), int(mean),
                                    dtype_code(G.dtype), G.shape[-1], _ptr(dZq), _stream()))


def sar_spmm_bwd_all(b: Blocks, G: torch.Tensor, mean: bool, dZq: Sequence[torch.Tensor]) -> None:
    native().spmm_bwd_all(b, G, mean, dZq)


def sar_error_add(Eq: Optional[torch.Tensor], t_rank: int, accumulate: bool, Ep: torch.Tensor) -> None:
    """t_rank: device address of the block's t_rank array (BlockView.t_rank)."""
    native().error_add(Eq, t_rank, accumulate, Ep)


# --------------------------------------------------------------------- GAT

def sar_gat_scores(Z: torch.Tensor, a: torch.Tensor, score: torch.Tensor) -> None:
    native().gat_scores(Z, a, score)


def sar_gat_fwd_begin(m: torch.Tensor, l: torch.Tensor, acc: torch.Tensor) -> None:
    native().gat_fwd_begin(m, l, acc)


def sar_gat_fwd_block(b: Blocks, q: int, Zq: torch.Tensor, s: torch.Tensor, tq: Optional[torch.Tensor],
                      a_l: Optional[torch.Tensor], slope: float,
                      m: torch.Tensor, l: torch.Tensor, acc: torch.Tensor) -> None:
    native().gat_fwd_block(b, q, Zq, s, tq, a_l, slope, m, l, acc)


def sar_gat_fwd_end(m: torch.Tensor, l: torch.Tensor, acc: torch.Tensor, out: torch.Tensor,
                    L: torch.Tensor, act: int = SAR_ACT_NONE) -> None:
    native().gat_fwd_end(m, l, acc, out, L, act)


def sar_gat_fwd_all(b: Blocks, Zq: Sequence[torch.Tensor], s: torch.Tensor,
                    tq: Optional[Sequence[torch.Tensor]], a_l: Optional[torch.Tensor],
                    slope: float, out: torch.Tensor, L: torch.Tensor, act: int = SAR_ACT_NONE) -> None:
    native().gat_fwd_all(b, Zq, s, tq, a_l, slope, out, L, act)


def sar_gat_workspace_bytes(n_dst: int, n_src_max: int, H: int, D: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().sar_gat_workspace_bytes(n_dst, n_src_max, H, D,
                                         ctypes.byref(out)))
    return out.value


def sar_gat_bwd_begin(G: torch.Tensor, out: torch.Tensor, s: torch.Tensor, L: torch.Tensor,
                      rec: torch.Tensor, ds: torch.Tensor, act: int = SAR_ACT_NONE,
                      Gact: Optional[torch.Tensor] = None) -> None:
    native().gat_bwd_begin(G, out, s, L, rec, ds, act, Gact)


def sar_gat_bwd_block(b: Blocks, q: int, Zq: torch.Tensor, G: torch.Tensor, tq: torch.Tensor,
                      rec: torch.Tensor, a_l: torch.Tensor, slope: float, dZq: torch.Tensor,
                      dtq: Optional[torch.Tensor], ds: torch.Tensor, da_l: torch.Tensor, work: torch.Tensor) -> None:
    """dtq None: the per-source sums dt_q are not written (dZq and da_l contain them already)."""
    native().gat_bwd_block(b, q, Zq, G, tq, rec, a_l, slope, dZq, dtq, ds, da_l, work)


def sar_gat_bwd_all(b: Blocks, Zq: Sequence[torch.Tensor], G: torch.Tensor, tq: Sequence[torch.Tensor],
                    rec: torch.Tensor, a_l: torch.Tensor, slope: float, dZq: Sequence[torch.Tensor],
                    dtq: Optional[Sequence[torch.Tensor]], ds: torch.Tensor, da_l: torch.Tensor,
                    work: torch.Tensor) -> None:
    """dtq None: the per-source sums dt_q are not written (dZq and da_l contain them already)."""
    native().gat_bwd_all(b, Zq, G, tq, rec, a_l, slope, dZq, dtq, ds, da_l, work)


def sar_gat_bwd_end(Zdst: torch.Tensor, ds: torch.Tensor, a_r: torch.Tensor, dZadd: Optional[torch.Tensor],
                    dZdst: Optional[torch.Tensor], da_r: torch.Tensor, work: torch.Tensor,
                    dZadd_rank: Optional[int] = None) -> None:
    """dZadd_rank: device address of the local block's t_rank (BlockView.t_rank) when dZadd is compact.
    dZdst None: only da_r."""
    native().gat_bwd_end(Zdst, ds, a_r, dZadd, dZdst, da_r, work, dZadd_rank)


def sar_gat_bwd_end_noalloc(Zdst: torch.Tensor, ds: torch.Tensor, a_r: torch.Tensor,
                            dZadd: Optional[torch.Tensor], dZdst: torch.Tensor, da_r: torch.Tensor,
                            dZadd_rank: Optional[int] = None) -> None:
    H, D = a_r.shape
    _check(lib().sar_gat_bwd_end_noalloc(_ptr(Zdst), _ptr(ds), _ptr(a_r), _ptr(dZadd), dZadd_rank, _ptr(dZdst), _ptr(da_r),
                                         dtype_code(Zdst.dtype), Zdst.shape[0], H,
                                         D, _stream()))


# ------------------------------------------------------------------ linear

def sar_linear_workspace_bytes(n: int, K: int, F: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().sar_linear_workspace_bytes(n, K, F, ctypes.byref(out)))
    return out.value


def sar_linear_fwd(X: torch.Tensor, W: torch.Tensor, Z: torch.Tensor,
                   a_score: Optional[torch.Tensor] = None, score: Optional[torch.Tensor] = None,
                   a_score2: Optional[torch.Tensor] = None, score2: Optional[torch.Tensor] = None) -> None:
    native().linear_fwd(X, W, Z, a_score, score, a_score2, score2)


def sar_linear_bwd(X: Optional[torch.Tensor], dZ: torch.Tensor, W: Optional[torch.Tensor],
                   dW: Optional[torch.Tensor], dX: Optional[torch.Tensor],
                   work: Optional[torch.Tensor]) -> None:
    native().linear_bwd(X, dZ, W, dW, dX, work)


def sar_linear_bwd_rows(X: Optional[torch.Tensor], E: Optional[torch.Tensor], E_rank: Optional[int],
                        ds: Optional[torch.Tensor], a_r: Optional[torch.Tensor], H: int, D: int,
                        W: Optional[torch.Tensor], dW: Optional[torch.Tensor], dX: Optional[torch.Tensor],
                        n: int, dtype: torch.dtype, work: Optional[torch.Tensor],
                        rows: Optional[torch.Tensor] = None) -> None:
    """E_rank: device address of a t_rank array (BlockView.t_rank) when E is compact."""
    native().linear_bwd_rows(X, E, E_rank, ds, a_r, H, D, W, dW, dX, n, dtype_code(dtype), work, rows)
