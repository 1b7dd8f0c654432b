"""The library's own rules for a launch's shape, by their C++ names (they are not part of the C ABI).  Not a test module."""
import ctypes

from paper_2503_05840_amd import binding


def _rule(name, restype, *argtypes):
    f = getattr(binding.load(), name)
    f.restype, f.argtypes = restype, argtypes
    return f


def batch_tiles(B, rows, e, units):
    """Batch tiles of 16 sequences that a workgroup of a product takes (units: heads, times matrices for a block's products)."""
    i = ctypes.c_int
    return _rule("_ZN4slim16proj_batch_tilesEiiii", i, i, i, i, i)(B, rows, e, units)


def batch_chunks(B, rows, e, units):
    per = 16 * batch_tiles(B, rows, e, units)
    return (B + per - 1) // per


def row_splits(units, rows, e, B):
    i = ctypes.c_int
    return _rule("_ZN4slim15proj_row_splitsEiiii", i, i, i, i, i)(units, rows, e, B)


def read_once(weight_bytes, cache_bytes):
    """Whether a call's loads of its weights are nontemporal, where one batch chunk reads a matrix."""
    return _rule("_ZN4slim9read_onceEmm", ctypes.c_bool, ctypes.c_size_t, ctypes.c_size_t)(weight_bytes, cache_bytes)


def xcache_read_once(B, T, d_model, e, ragged, one_pass):
    i, b = ctypes.c_int, ctypes.c_bool
    return _rule("_ZN4slim16xcache_read_onceEiiiibb", b, i, i, i, i, b, b)(B, T, d_model, e, ragged, one_pass)


class _Cut(ctypes.Structure):
    _fields_ = [("tiles", ctypes.c_int), ("splits", ctypes.c_int)]


def one_pass_cut(B, H, T, d_model, ragged=False):
    """Head tiles of a workgroup of the one-pass X-cache kernel, context splits, and the most that any context up to T takes."""
    i, b = ctypes.c_int, ctypes.c_bool
    most = _rule("_ZN4slim18xfused_most_splitsEiiii", i, i, i, i, i)(B, H, T, d_model)
    cut = _rule("_ZN4slim10xfused_cutEiiiibi", _Cut, i, i, i, i, b, i)(B, H, T, d_model, ragged, most)
    return cut.tiles, cut.splits, most


def one_pass_splits(B, H, T, d_model, ragged=False):
    return one_pass_cut(B, H, T, d_model, ragged)[1:]


def one_pass_through(nbytes):
    """Whether that many bytes of the one-pass X-cache kernel's partials leave through the L2s."""
    return _rule("_ZN4slim14xfused_throughEm", ctypes.c_bool, ctypes.c_size_t)(nbytes)
