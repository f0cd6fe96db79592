"""Which kernel a shape takes, asked of the library's own rules: the GPU tests of
a kernel call these, so that a change of a rule cannot lead their shapes past
the kernel unseen."""

import ctypes

from paper_2402_00518_amd import binding as B


def _rule(symbol, *types):
    f = getattr(ctypes.CDLL(B.LIB_PATH), symbol)
    f.restype, f.argtypes = ctypes.c_bool, types
    return f


def mid_tile(big_tiles):
    """Do bf16 products with this many 256 x 256 tiles take 128 x 128 ones?"""
    return _rule("_ZN2ee13gemm_mid_tileEl", ctypes.c_int64)(big_tiles)


def f32_small(tiles, small_tiles, k):
    """Do fp32 products with these counts of 128 x 128 and 64 x 64 tiles take the latter?"""
    f = ctypes.CDLL(B.LIB_PATH)["_ZN2ee14gemm_f32_smallElli"]
    f.restype, f.argtypes = ctypes.c_bool, (ctypes.c_int64, ctypes.c_int64, ctypes.c_int)
    return f(tiles, small_tiles, k)


def f32_parts(tiles, small_tiles):
    """Parts in which 128 x 128 fp32 tiles sum K."""
    f = ctypes.CDLL(B.LIB_PATH)["_ZN2ee14gemm_f32_partsEll"]
    f.restype, f.argtypes = ctypes.c_int, (ctypes.c_int64, ctypes.c_int64)
    return f(tiles, small_tiles)


def f32_loops(tiles):
    """Does a launch of this many 128 x 128 fp32 tiles loop over them?"""
    return _rule("_ZN2ee14gemm_f32_loopsEl", ctypes.c_int64)(tiles)


def gsum_rows(f32, ldn, vocab):
    """Rows of the logit gradient that a block of the row-sum kernel takes."""
    f = ctypes.CDLL(B.LIB_PATH)["_ZN2ee9gsum_rowsEbii"]
    f.restype, f.argtypes = ctypes.c_int, (ctypes.c_bool, ctypes.c_int, ctypes.c_int)
    return f(f32, ldn, vocab)


class _SplitTail(ctypes.Structure):
    _fields_ = [("tok0", ctypes.c_int), ("feat0", ctypes.c_int), ("splits", ctypes.c_int)]


def split_tail(f32, n, h, k, most=4):
    """Split of an n x h product over k: (first split token, first split feature, slices)."""
    f = ctypes.CDLL(B.LIB_PATH)["_ZN2ee10split_tailEbiiii"]
    f.restype, f.argtypes = _SplitTail, (ctypes.c_bool,) + (ctypes.c_int,) * 4
    s = f(f32, n, h, k, most)
    return s.tok0, s.feat0, s.splits


_INT3 = (ctypes.c_int,) * 3


def skinny_logits(rows, n, k):
    return _rule("_ZN2ee20decode_skinny_logitsEiii", *_INT3)(rows, n, k)


def skinny_down(rows, n, k):
    return _rule("_ZN2ee18decode_skinny_downEiii", *_INT3)(rows, n, k)
