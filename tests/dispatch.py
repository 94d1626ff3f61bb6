"""The library's own answers to which kernel a call takes: host functions of libsasq.so, no device needed."""
from __future__ import annotations

import ctypes

from paper_2512_14481_amd import binding as B


def _function(symbol, *argtypes):
    f = getattr(B._lib(), symbol)
    f.restype, f.argtypes = ctypes.c_int, argtypes
    return f


def bwd_rows(M, N, K):
    """Rows per workgroup of the backward linear's few-row and row-block kernels, 0: the GEMM's tiles (sasq::bwd_rows)."""
    i64 = ctypes.c_int64
    return _function("_ZN4sasq8bwd_rowsElll", i64, i64, i64)(M, N, K)


def bwd_turns(M, N, K):
    """Whether dY turns in LDS in the backward linear's few-row and row-block kernels (sasq::bwd_turns)."""
    i64 = ctypes.c_int64
    return bool(_function("_ZN4sasq9bwd_turnsElll", i64, i64, i64)(M, N, K) & 1)


def bwd_tile(M, N, K):
    """The backward GEMM's tile, rows and columns (sasq::bwd_tile)."""
    i64 = ctypes.c_int64
    return ((256, 256), (128, 256), (128, 128))[_function("_ZN4sasq8bwd_tileElll", i64, i64, i64)(M, N, K)]


def bwd_reads_lines(N, tile_rows):
    """Whether the backward GEMM's tiles of so many rows read dY in whole cache lines (sasq::bwd_reads_lines)."""
    return bool(_function("_ZN4sasq15bwd_reads_linesEli", ctypes.c_int64, ctypes.c_int)(N, tile_rows) & 1)


def grouped_form(M, N, K, group, blocked):
    """The form of the grouped linear's split kernel, 0: the other kernels (sasq::grouped_takes_split)."""
    i64 = ctypes.c_int64
    return _function("_ZN4sasq19grouped_takes_splitEllllb", i64, i64, i64, i64, ctypes.c_bool)(M, N, K, group, blocked)


def anyk_few_rows(M, N, K):
    """Whether a static linear with K not a multiple of 64 takes the few-row kernel (sasq::linear_anyk_takes_skinny)."""
    i64 = ctypes.c_int64
    return bool(_function("_ZN4sasq24linear_anyk_takes_skinnyElll", i64, i64, i64)(M, N, K) & 1)


ANYK_TILES = ((256, 128, 8), (128, 128, 8), (128, 128, 4), (64, 128, 8), (64, 128, 4), (64, 64, 4), (32, 64, 4))


def anyk_tile(M, N, K):
    """The tile of a linear with K not a multiple of 64 and more rows: rows, columns, waves (sasq::linear_anyk_tile)."""
    i64 = ctypes.c_int64
    return ANYK_TILES[_function("_ZN4sasq16linear_anyk_tileElll", i64, i64, i64)(M, N, K)]


class _LinItem(ctypes.Structure):
    _fields_ = [(f, ctypes.c_void_p) for f in ("x", "xq", "s", "wq", "s_w", "bias", "y")] + [(f, ctypes.c_int) for f in ("M", "N", "K", "tiles_m", "tiles_n")]


class _LinBatch(ctypes.Structure):
    _fields_ = [("it", _LinItem * 8), ("first_block", ctypes.c_int * 9)] + [(f, ctypes.c_int) for f in ("count", "split_first", "split_count", "trim_rows")]


def _batch(items):
    batch = _LinBatch(count=len(items))
    for i, (m, n, k) in enumerate(items):
        batch.it[i].M, batch.it[i].N, batch.it[i].K = m, n, k
    return ctypes.byref(batch)


def linear_block_rows(items, wf):
    """Rows per workgroup of the linear's row blocks for (rows, columns, K) items of more than 64 rows, 32: small blocks, 0: the GEMM's
    tiles (sasq::linear_block_rows)."""
    return _function("_ZN4sasq17linear_block_rowsERKNS_8LinBatchEi", ctypes.POINTER(_LinBatch), ctypes.c_int)(_batch(items), wf)


def linear_takes_few_rows(items, wf):
    """Whether the items take the few-row, small-block or row-block kernels (sasq::linear_takes_skinny)."""
    return bool(_function("_ZN4sasq19linear_takes_skinnyERKNS_8LinBatchEi", ctypes.POINTER(_LinBatch), ctypes.c_int)(_batch(items), wf) & 1)


def linear_quantizes(items, wf):
    """Whether such a call quantizes the activations in the kernel (sasq::linear_quantizes_in_kernel)."""
    f = _function("_ZN4sasq26linear_quantizes_in_kernelERKNS_8LinBatchEib", ctypes.POINTER(_LinBatch), ctypes.c_int, ctypes.c_bool)
    return bool(f(_batch(items), wf, False) & 1)


def linear_streams(items, wf):
    """Whether such a call reads its weights past the caches (sasq::linear_streams)."""
    return bool(_function("_ZN4sasq14linear_streamsERKNS_8LinBatchEi", ctypes.POINTER(_LinBatch), ctypes.c_int)(_batch(items), wf) & 1)


def linear_long_rows(items):
    """Whether the wide few-row form keeps six K tiles a wave in flight (sasq::linear_long_rows)."""
    return bool(_function("_ZN4sasq16linear_long_rowsERKNS_8LinBatchE", ctypes.POINTER(_LinBatch))(_batch(items)) & 1)


def linear_turns(items, wf):
    """Whether the operands of a few-row, small-block or row-block call turn in LDS, as it quantizes in the kernel or not (sasq::linear_turns)."""
    f = _function("_ZN4sasq12linear_turnsERKNS_8LinBatchEib", ctypes.POINTER(_LinBatch), ctypes.c_int, ctypes.c_bool)
    return bool(f(_batch(items), wf, linear_quantizes(items, wf)) & 1)
