"""The library's launch rules and tile shapes as its tests see them (the mxt_
entry points of libmxnorm.so)."""
import ctypes

import torch

from paper_2603_13180_amd import mxnorm

SHAPES = ["k16x32", "k32x32", "k32x64", "k64x64", "r64x128", "r128x128", "t256x256"]
PAIRS = ["apart", "large", "small"]
ELEM = {"e4m3": 0, "e2m1": 1}
UNITS = 256                                            # compute units of an MI355X

_I, _L, _D, _P = ctypes.c_int, ctypes.c_int64, ctypes.c_double, ctypes.c_void_p


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


def matmul_as(ac, as_, bc, bs, K, elem, shape, whole=0, units=0, out=None, b_gain=None,
              out_dtype=torch.float32):
    """mx_matmul_fwd in tiles of `shape` (or `whole` cells of 256 x 256 first),
    the persistent kernels as on `units` compute units; GPU tensors."""
    M, N = ac.shape[0], bc.shape[0]
    if out is None:
        out = torch.empty(M, N, dtype=out_dtype, device=ac.device)
    f = _fn("mxt_matmul", [_P] * 4 + [_L] * 3 + [_I, _P, _I, _P, _I, _I, _I, _P])
    mxnorm._check(f(ac.data_ptr(), as_.data_ptr(), bc.data_ptr(), bs.data_ptr(), M, N, K, ELEM[elem],
                    None if b_gain is None else b_gain.data_ptr(), mxnorm.OUT_DTYPES[out.dtype],
                    out.data_ptr(), SHAPES.index(shape), whole, units, mxnorm._stream(ac.device)))
    return out


class _Product(ctypes.Structure):
    _fields_ = [(n, _P) for n in ("a", "as_", "b", "bs")] + [(n, _L) for n in "MNK"] + \
        [("gain", _P), ("out", _P)]


def matmul_pair_as(f32, bf16, elem, mode, units=0):
    """Two products at once; each (a codes, a scales, b codes, b scales, K,
    gain or None, out)."""
    def product(a, as_, b, bs, K, gain, out):
        return _Product(a.data_ptr(), as_.data_ptr(), b.data_ptr(), bs.data_ptr(), a.shape[0],
                        b.shape[0], K, None if gain is None else gain.data_ptr(), out.data_ptr())
    f = _fn("mxt_matmul_pair", [_P, _P, _I, _I, _I, _P])
    mxnorm._check(f(ctypes.byref(product(*f32)), ctypes.byref(product(*bf16)), ELEM[elem],
                    PAIRS.index(mode), units, mxnorm._stream(f32[0].device)))
