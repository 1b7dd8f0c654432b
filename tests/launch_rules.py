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


def one_pass_splits(B, H, T, d_model):
    """Context splits of the one-pass X-cache kernel, and the most that any context up to T takes."""
    i = ctypes.c_int
    return tuple(_rule("_ZN4slim%sEiiii" % name, i, i, i, i, i)(B, H, T, d_model) for name in ("13xfused_splits", "18xfused_most_splits"))


def one_pass_through(nbytes):
    """Whether that many bytes of the one-pass X-cache kernel's partials leave through the L2s."""
    return _rule("_ZN4slim14xfused_throughEm", ctypes.c_bool, ctypes.c_size_t)(nbytes)


def one_pass_tiles(B, H, T, d_model):
    """Head tiles of a workgroup of the one-pass X-cache kernel."""
    i = ctypes.c_int
    return _rule("_ZN4slim12xfused_tilesEiiii", i, i, i, i, i)(B, H, d_model, one_pass_splits(B, H, T, d_model)[0])
