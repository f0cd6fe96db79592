"""Which kernel a shape takes, asked of the library's own rules: the GPU tests of
a kernel call these, so that a change of a rule cannot lead their shapes past
the kernel unseen."""

import ctypes

from paper_2402_00518_amd import binding as B


def _rule(symbol, *types):
    f = getattr(ctypes.CDLL(B.LIB_PATH), symbol)
    f.restype, f.argtypes = ctypes.c_bool, types
    return f


_INT3 = (ctypes.c_int,) * 3


def skinny_logits(rows, n, k):
    return _rule("_ZN2ee20decode_skinny_logitsEiii", *_INT3)(rows, n, k)


def skinny_down(rows, n, k):
    return _rule("_ZN2ee18decode_skinny_downEiii", *_INT3)(rows, n, k)
