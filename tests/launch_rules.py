"""The library's launch rules and tile shapes as its tests see them (the mxt_
entry points of libmxnorm.so)."""
import ctypes

from paper_2603_13180_amd import mxnorm

SHAPES = ["k16x32", "k32x32", "k32x64", "k64x64", "r64x128", "r128x128", "t256x256"]
PAIRS = ["apart", "large", "small"]
ELEM = {"e4m3": 0, "e2m1": 1}
UNITS = 256                                            # compute units of an MI355X

_I, _L, _D = ctypes.c_int, ctypes.c_int64, ctypes.c_double


def _fn(name, args):
    f = getattr(mxnorm.load(), name)
    f.restype, f.argtypes = _I, args
    return f


def norm_team(T, d, kind, fmt, gain):
    return _fn("mxt_norm_team", [_L, _L, _I, _I, _I])(T, d, kind, fmt, gain)


def product_plan(M, N, K, elem, units=UNITS):
    """(tile shape, 256 x 256 cells of a first launch, shape of the second, us)"""
    whole, tail, us = _I(), _I(), _D()
    f = _fn("mxt_product_plan", [_L, _L, _L, _I, _I] + [ctypes.c_void_p] * 3)
    s = f(M, N, K, ELEM[elem], units, ctypes.byref(whole), ctypes.byref(tail), ctypes.byref(us))
    assert s >= 0, (M, N, K, elem)
    return SHAPES[s], whole.value, SHAPES[tail.value] if whole.value else None, us.value


def shape_of(M, N, K, elem, units=UNITS):
    """The tile shape, or "t256x256+<tail>"."""
    s, whole, tail, _ = product_plan(M, N, K, elem, units)
    return s + "+" + tail if whole else s


def pair_plan(T, N, d, elem, units=UNITS):
    """(how the backward computes its products, [us apart, large, small])"""
    us = (_D * 3)()
    m = _fn("mxt_pair_plan", [_L] * 6 + [_I, _I, ctypes.c_void_p])(N, d, T, T, d, N, ELEM[elem],
                                                                  units, us)
    assert m >= 0, (T, N, d, elem)
    return PAIRS[m], list(us)
