"""Every product kernel against the oracle, at sizes the oracle can check in
full.

mx_matmul_fwd chooses a tile shape by an estimate of its time, so a size says
nothing lasting about the kernel that runs it.  These tests name the kernel:
each tile shape alone, 256 x 256 cells followed by each smaller shape over the
rest, and the backward's two products in each kind of launch.  The persistent
kernels run as on a few compute units, so that a workgroup goes from whole and
partial tiles to the next one.  Outputs lie in a buffer whose last elements
show a store past the end."""
import functools

import numpy as np
import pytest
import torch

import launch_rules
import oracle
from launch_rules import SHAPES, matmul_as, matmul_pair_as
from paper_2603_13180_amd import mxnorm
from test_gpu_gemm import (abs_codes, assert_close, dev_u8, one_hot_operand, oracle_product,
                           random_operand)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ELEMS = ["e4m3", "e2m1"]
DTYPES = [torch.float32, torch.bfloat16]
SMALLER = SHAPES[:-1]

# (tile shape, 256 x 256 cells before it, compute units; 0: the device's)
WAYS = [(s, 0, 0) for s in SHAPES] + \
    [(s, 0, u) for s in ("r64x128", "r128x128", "t256x256") for u in (1, 2)] + \
    [(s, 3, 0) for s in SMALLER] + [("r64x128", 2, 1), ("r128x128", 2, 2)]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        raise RuntimeError("GPU tile tests need a GPU (run them with -m gpu on an MI355X)")
    mxnorm.load()


def guarded(M, N, dtype):
    buf = torch.full((M * N + 64,), 7.0, dtype=dtype, device=DEV)
    return buf, buf[:M * N].view(M, N)


def host(h):
    return h.float().cpu().numpy().astype(np.float64)


def rounded(want, dtype):
    """One exact float32 product per output, in the output's type."""
    w32 = want.astype(np.float32)
    assert np.array_equal(w32.astype(np.float64), want)
    if dtype == torch.bfloat16:
        w32 = torch.from_numpy(w32).to(torch.bfloat16).float().numpy()
    return w32.astype(np.float64)


@functools.lru_cache(maxsize=None)
def one_hot_case(elem, M=640, N=528, K=512):
    rng = np.random.default_rng(5)
    ac, as_ = one_hot_operand(M, K, elem, np.arange(M) % K, rng)
    bc, bs = one_hot_operand(N, K, elem, (np.arange(N) * 7) % K, rng)
    want = oracle.mx_matmul(ac, as_, bc, bs, K, elem=elem)
    assert (want != 0).sum() >= M // 8
    return [dev_u8(v) for v in (ac, as_, bc, bs)], want, K


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("elem", ELEMS)
@pytest.mark.parametrize("shape,whole,units", WAYS)
def test_single_products_are_exact(elem, shape, whole, units, dtype):
    # at most one product per output, exact in float32: every k of 512, every
    # scale block and every output column is pinned bit for bit.  640 x 528 is
    # 3 x 3 cells, the last 128 rows and 16 columns of them partial
    t, want, K = one_hot_case(elem)
    buf, h = guarded(*want.shape, dtype)
    matmul_as(*t, K, elem, shape, whole, units, out=h)
    assert (buf[h.numel():] == 7.0).all()
    got, want = host(h), rounded(want, dtype)
    bad = np.argwhere(got != want)
    assert bad.size == 0, "%d outputs differ, first %s: got %r want %r" % (
        len(bad), bad[0], got[tuple(bad[0])], want[tuple(bad[0])])


@functools.lru_cache(maxsize=None)
def random_case(elem, M, N, K, special=False):
    rng = np.random.default_rng(M + 3 * N + 5 * K + len(elem))
    ac, as_ = random_operand(M, K, elem, rng)
    bc, bs = random_operand(N, K, elem, rng)
    if special:
        as_[3, 5] = as_[M - 1, 0] = 0xFF        # rows of NaN
        bs[17, 0] = bs[N - 1, K // 32 - 1] = 0xFF
        if elem == "e4m3":
            ac[M // 2, K - 1] = 0x7F
    want, mag = oracle_product(ac, as_, bc, bs, K, elem)
    gain = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).to(torch.bfloat16)
    return [dev_u8(v) for v in (ac, as_, bc, bs)], want, mag, gain


def check(h, want, mag, gain, ctx):
    f = 1.0 if gain is None else gain.double().numpy()
    # the gain's product rounds once more in float32
    extra = 0.0 if gain is None else 2.0 ** -23 * np.abs(want * f)
    assert_close(host(h), want * f, mag * np.abs(f) + 2.0 ** 9 * extra, h.dtype == torch.bfloat16, ctx)


@pytest.mark.parametrize("elem", ELEMS)
@pytest.mark.parametrize("shape,whole,units", WAYS)
def test_nan_scales_and_codes_propagate(elem, shape, whole, units):
    M, N, K = 300, 528, 512
    t, want, mag, _ = random_case(elem, M, N, K, special=True)
    assert np.isnan(want[[3, M - 1]]).all() and np.isnan(want[:, [17, N - 1]]).all()
    for dtype in DTYPES:
        h = matmul_as(*t, K, elem, shape, whole, units, out_dtype=dtype)
        check(h, want, mag, None, "nan %s %s %d %d" % (elem, shape, whole, units))


# 531 x 560: 3 x 3 cells, remainders in every tile shape; 10 or 5 K steps: a
# ring's slots come round several times, and K-split waves have one step or two
@pytest.mark.parametrize("elem", ELEMS)
@pytest.mark.parametrize("shape,whole,units", WAYS)
def test_every_output(elem, shape, whole, units):
    M, N, K = 531, 560, 1280
    t, want, mag, gain = random_case(elem, M, N, K)
    for dtype in DTYPES:
        for g in (None, gain):
            buf, h = guarded(M, N, dtype)
            matmul_as(*t, K, elem, shape, whole, units, out=h, b_gain=None if g is None else g.to(DEV))
            assert (buf[M * N:] == 7.0).all()
            check(h, want, mag, g, "%s %s %d %d" % (elem, shape, whole, units))


@pytest.mark.parametrize("elem", ELEMS)
def test_only_k_split_changes_the_order_of_additions(elem):
    # rings, 256 x 256 tiles, tails and pairs add the K steps in order: the same
    # bits; K-split tiles add eight partial sums, the same for all of them
    M, N, K = 531, 560, 2560
    t, _, _, _ = random_case(elem, M, N, K)
    bits = {}
    for shape, whole, units in WAYS:
        if not whole:
            bits[shape, units] = matmul_as(*t, K, elem, shape, 0, units)
    want = bits["t256x256", 0]
    split = bits["k64x64", 0]
    assert not torch.equal(split, want)
    for (shape, units), h in bits.items():
        assert torch.equal(h, split if shape.startswith("k") else want), (shape, units)
    for mode in ("large", "small"):
        outs = [torch.empty(M, N, device=DEV), torch.empty(M, N, dtype=torch.bfloat16, device=DEV)]
        matmul_pair_as(*[(*t, K, None, o) for o in outs], elem, mode)
        assert torch.equal(outs[0], want) and torch.equal(outs[1], want.to(torch.bfloat16))


@pytest.mark.parametrize("elem", ELEMS)
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("M,N,K", [(1, 16, 256), (257, 272, 256), (129, 144, 2816)])
def test_smallest_and_uneven(elem, shape, M, N, K):
    # fewer K steps than waves or ring slots, one row, one column group, and
    # a step count that no wave count divides
    t, want, mag, _ = random_case(elem, M, N, K)
    buf, h = guarded(M, N, torch.bfloat16)
    matmul_as(*t, K, elem, shape, out=h)
    assert (buf[M * N:] == 7.0).all()
    check(h, want, mag, None, "%s %s" % (elem, shape))


@pytest.mark.parametrize("units", [8, 0])
@pytest.mark.parametrize("elem", ELEMS)
def test_256_tiles_in_groups_every_output(elem, units):
    # 9 tile rows (two full groups of 4 and a group of 1) x 5 tile columns (the
    # last one 16 columns wide), K = 4096; on 8 units a workgroup computes up
    # to 6 of the 45 tiles, partial ones followed by whole ones
    M, N, K = 2304, 1040, 4096
    t, want, mag, _ = random_case(elem, M, N, K)
    for dtype in DTYPES:
        h = matmul_as(*t, K, elem, "t256x256", units=units, out_dtype=dtype)
        check(h, want, mag, None, "256 x 256 %s" % elem)


# ------------------------------------------------ two products, one launch --

PAIR_WAYS = [("large", 0), ("large", 16), ("large", 8), ("large", 1), ("small", 0), ("apart", 0)]
# products of 9 and 8 cells; the longer K first and second
PAIR_SIZES = [((531, 560, 1280), (777, 304, 768)), ((531, 560, 768), (777, 304, 1280))]


@pytest.mark.parametrize("elem", ELEMS)
@pytest.mark.parametrize("sizes", PAIR_SIZES)
@pytest.mark.parametrize("mode,units", PAIR_WAYS)
def test_pairs_every_output(elem, sizes, mode, units):
    cases = [random_case(elem, *s, special=i == 1) for i, s in enumerate(sizes)]
    for gains in ((False, False), (True, False)):
        outs = [guarded(s[0], s[1], dt) for s, dt in zip(sizes, DTYPES)]
        g = [c[3] if on else None for c, on in zip(cases, gains)]
        matmul_pair_as(*[(*c[0], s[2], None if gi is None else gi.to(DEV), o[1])
                         for c, s, gi, o in zip(cases, sizes, g, outs)], elem, mode, units)
        for i, ((buf, h), c) in enumerate(zip(outs, cases)):
            assert (buf[h.numel():] == 7.0).all()
            check(h, c[1], c[2], g[i], "pair %s %s %d product %d" % (elem, mode, units, i))


@pytest.mark.parametrize("elem", ELEMS)
@pytest.mark.parametrize("mode,units", PAIR_WAYS)
def test_pairs_of_single_products_are_exact(elem, mode, units):
    c0, c1 = one_hot_case(elem), one_hot_case(elem, 528, 640, 512)
    outs = [guarded(*c[1].shape, dt) for c, dt in zip((c0, c1), DTYPES)]
    matmul_pair_as(*[(*c[0], c[2], None, o[1]) for c, o in zip((c0, c1), outs)], elem, mode, units)
    for (buf, h), c, dt in zip(outs, (c0, c1), DTYPES):
        assert (buf[h.numel():] == 7.0).all()
        assert np.array_equal(host(h), rounded(c[1], dt)), (mode, units, dt)


def test_unknown_ways_are_refused():
    t, _, K = one_hot_case("e4m3")
    for kw in (dict(whole=9), dict(whole=-1), dict(units=-1), dict(units=1 << 20)):
        with pytest.raises(mxnorm.MXNormError):
            matmul_as(*t, K, "e4m3", "r64x128", **kw)
    assert launch_rules.shape_of(640, 528, 512, "e4m3") in SHAPES
