"""GPU parity of the MXNormLinear backward pieces against the oracle (Sec.
3.7; the RMSNorm-gradient appendix; the implementation appendix's
mx_norm_linear_backward): the column-wise MX cast (bit-exact), the
straight-through estimator (within bounds derived from its float
arithmetic), the matmul's column gain, and the whole backward composed from
the library's kernels, checked stage by stage."""
import numpy as np
import pytest
import torch

import launch_rules
import oracle
from paper_2603_13180_amd import mxnorm, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        raise RuntimeError("GPU backward tests need a GPU (run them with -m gpu on an MI355X)")
    mxnorm.load()


def dev_bf16(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(DEV).view(torch.bfloat16)


def bits_of(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def f64(bits):
    return synth.bf16_bits_to_f32(bits).astype(np.float64)


# ----------------------------------------------------------- column cast --

def check_cast_t(xb, rho, elem, mode):
    x = dev_bf16(xb)
    r = None if rho is None else torch.from_numpy(rho).to(DEV)
    codes, scales = mxnorm.mx_cast_t_fwd(x, r, elem=elem, scale_mode=mode)
    torch.cuda.synchronize()
    wc, ws = oracle.mxcast_t(xb, rho, B=32, elem=elem, mode=mode)
    ctx = "cast_t %s %s %s rho=%s" % (xb.shape, elem, mode, rho is not None)
    s, c = scales.cpu().numpy(), codes.cpu().numpy()
    bad = np.argwhere(s != ws)
    assert bad.size == 0, "%s: %d scale bytes differ, first %s" % (ctx, len(bad), bad[0])
    bad = np.argwhere(c != wc)
    assert bad.size == 0, "%s: %d codes differ, first %s got %#x want %#x" % (
        ctx, len(bad), bad[0], c[tuple(bad[0])], wc[tuple(bad[0])])


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
@pytest.mark.parametrize("R,C", [(32, 8), (96, 40), (160, 200), (256, 64), (1024, 1000),
                                 (4096, 256), (64, 8200), (288, 8448), (160, 12296)])
def test_cast_t_shapes(elem, R, C):
    # ragged last column tiles (8200, 8448, 12296) and row tiles (160, 288);
    # from 48 column tiles (12288 columns) on the workgroups visit the tiles
    # in XCD ranges of 64-row-tile groups (12296 x 160: one partial group)
    xb = synth.gaussian(R, C, seed=R + C, scale=2.0)
    rho = np.random.default_rng(R).uniform(0.01, 8.0, R).astype(np.float32)
    for mode in ("rceil", "floor"):
        check_cast_t(xb, None, elem, mode)
        check_cast_t(xb, rho, elem, mode)


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
def test_cast_t_edge_columns(elem):
    # the forward's adversarial rows, laid out as columns (one per row of it)
    from test_gpu_parity import adversarial_rows
    for R in (64, 1024):
        xb = np.ascontiguousarray(adversarial_rows(R, seed=R).T)   # [R, 14] -> pad to 16 cols
        xb = np.ascontiguousarray(np.concatenate([xb, xb[:, :2]], axis=1))
        rho = np.full(R, 0.75, np.float32)
        for mode in ("rceil", "floor"):
            check_cast_t(xb, None, elem, mode)
            check_cast_t(xb, rho, elem, mode)


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
@pytest.mark.parametrize("R,C", [(16384, 4096), (32768, 4096), (4096, 28672), (16384, 16384),
                                 (8320, 12288)])
def test_cast_t_multi_tile_spans_sampled(elem, R, C):
    """Large shapes: the bench's [32768, 4096], the wide grad_H of the
    gate+up projection at 4096 tokens (112 column tiles, one partial group
    of row tiles in the XCD-range order), [16384, 16384] (two full groups)
    and [8320, 12288] (a full group and a partial one): output rows of sampled columns -- the first and last of column
    tiles and random ones -- against the oracle's cast of those columns
    alone (an output row depends only on its column and rho)."""
    rng = np.random.default_rng(R + C)
    xb = synth.gaussian(R, C, seed=C, scale=3.0)
    rho = rng.uniform(0.01, 8.0, R).astype(np.float32)
    cols = np.unique(np.concatenate([[0, 1, 63, 64, 127, 128, 255, 256, C - 64, C - 1],
                                     rng.choice(C, 24, replace=False)]))
    x = dev_bf16(xb)
    codes, scales = mxnorm.mx_cast_t_fwd(x, torch.from_numpy(rho).to(DEV), elem=elem)
    torch.cuda.synchronize()
    c, sc = codes.cpu().numpy(), scales.cpu().numpy()
    # the oracle casts a column block of 8 (its C must be a multiple of 8)
    for c0 in np.unique(cols // 8 * 8):
        wc, ws = oracle.mxcast_t(np.ascontiguousarray(xb[:, c0:c0 + 8]), rho, B=32, elem=elem,
                                 mode="rceil")
        assert np.array_equal(sc[c0:c0 + 8], ws), "cast_t [%d, %d] %s scales, cols %d.." % (
            R, C, elem, c0)
        assert np.array_equal(c[c0:c0 + 8], wc), "cast_t [%d, %d] %s codes, cols %d.." % (
            R, C, elem, c0)


def test_cast_t_empty():
    x = torch.empty(0, 64, dtype=torch.bfloat16, device=DEV)
    c, s = mxnorm.mx_cast_t_fwd(x)
    assert c.shape == (64, 0) and s.shape == (64, 0)


# ------------------------------------------------------------------- STE --

def ste_bounds(xb, gzb, gb, rho):
    """Size of the two terms of grad_x per element, and of the grad_gamma sum."""
    x, gz = f64(xb), f64(gzb)
    g = f64(gb) if gb is not None else np.ones(x.shape[1])
    r = rho.astype(np.float64)[:, None]
    dxb = gz * g
    u = np.sum(dxb * x, axis=1, keepdims=True)
    c = r ** 3 * u / x.shape[1]
    return np.abs(r * dxb) + np.abs(c * x), np.sum(np.abs(r * x * gz), axis=0)


def check_ste(T, d, gamma, out_dtype, want_gg, seed=0, xb=None):
    rng = np.random.default_rng(seed + T + d)
    if xb is None:
        xb = synth.gaussian(T, d, seed=seed + d, scale=1.5)
    gzb = synth.gaussian(T, d, seed=seed + d + 1, scale=0.2)
    gb = synth.f32_to_bf16_bits(rng.uniform(0.3, 2.0, d).astype(np.float32)) if gamma else None
    rho = rng.uniform(0.2, 3.0, T).astype(np.float32)
    gx, gg = mxnorm.mxnorm_ste_bwd(dev_bf16(xb), dev_bf16(gzb),
                                   None if gb is None else dev_bf16(gb),
                                   torch.from_numpy(rho).to(DEV), out_dtype=out_dtype,
                                   want_grad_gamma=want_gg)
    torch.cuda.synchronize()
    wx, wg = oracle.ste_bwd(xb, gzb, gb, rho)
    terms, gsum = ste_bounds(xb, gzb, gb, rho)
    got = gx.float().cpu().numpy().astype(np.float64)
    # float arithmetic: RN(rho dXb), RN(c x) with c rounded once, their
    # difference rounded: within 2^-21 of the terms plus 2^-22 of the result;
    # bf16 output adds half an ulp (2^-8 relative)
    tol = 2.0 ** -21 * terms + 2.0 ** -22 * np.abs(wx) + 1e-37
    if out_dtype == torch.bfloat16:
        tol = tol + 2.0 ** -8 * np.abs(wx)
    fin = np.isfinite(wx)
    err = np.abs(got - wx)
    bad = fin & (err > tol)
    ctx = "ste T=%d d=%d gamma=%s %s" % (T, d, gamma, out_dtype)
    assert not bad.any(), "%s: %d grad_x off, first %s got %r want %r" % (
        ctx, bad.sum(), np.argwhere(bad)[0], got[tuple(np.argwhere(bad)[0])],
        wx[tuple(np.argwhere(bad)[0])])
    if want_gg:
        # float partial sums over 32 rows (each term rounded twice), then a
        # double sum: within 2^-16 of sum |terms|
        g = gg.cpu().numpy().astype(np.float64)
        assert (np.abs(g - wg) <= 2.0 ** -16 * gsum + 1e-37).all(), ctx + ": grad_gamma"
    else:
        assert gg is None


@pytest.mark.parametrize("T,d", [(1, 8), (33, 64), (100, 1024), (40, 4096), (65, 2048),
                                 (9, 10240), (3, 32768), (70, 2056), (2049, 256), (4100, 512)])
def test_ste_shapes(T, d):
    check_ste(T, d, True, torch.bfloat16, True)
    check_ste(T, d, False, torch.float32, True)


def test_ste_bench_shape():
    # the bench's [32768, 4096]: 64 rows per workgroup (512 workgroups), the
    # three-set row pipeline run to its end, every element of grad_x and
    # grad_gamma compared
    check_ste(32768, 4096, True, torch.bfloat16, True, seed=3)


@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("gamma", [True, False])
@pytest.mark.parametrize("want_gg", [True, False])
def test_ste_options(out_dtype, gamma, want_gg):
    check_ste(77, 4096, gamma, out_dtype, want_gg, seed=5)


def test_ste_zero_and_constant_rows():
    T, d = 40, 512
    xb = synth.gaussian(T, d, seed=9)
    xb[3] = 0
    xb[7] = synth.f32_to_bf16_bits(np.full(d, -1.25, np.float32))
    check_ste(T, d, True, torch.float32, True, xb=xb)


def test_ste_deterministic_and_workspace_reuse():
    T, d = 300, 4096
    xb = synth.gaussian(T, d, seed=1)
    gzb = synth.gaussian(T, d, seed=2)
    x, gz = dev_bf16(xb), dev_bf16(gzb)
    rho = torch.rand(T, device=DEV) + 0.5
    ws = torch.empty(mxnorm.load().mxnorm_ste_bwd_workspace_bytes(T, d), dtype=torch.uint8,
                     device=DEV)
    a = mxnorm.mxnorm_ste_bwd(x, gz, None, rho, workspace=ws)
    b = mxnorm.mxnorm_ste_bwd(x, gz, None, rho, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


# ---------------------------------------------------- matmul column gain --

@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
def test_matmul_column_gain(elem):
    from test_gpu_gemm import random_operand, abs_codes, assert_close
    M, N, K = 130, 272, 512
    rng = np.random.default_rng(3)
    ac, as_ = random_operand(M, K, elem, rng)
    bc, bs = random_operand(N, K, elem, rng)
    gb = synth.f32_to_bf16_bits(rng.uniform(-2, 2, N).astype(np.float32))
    t = [torch.from_numpy(v).to(DEV) for v in (ac, as_, bc, bs)]
    h = mxnorm.mx_matmul_fwd(*t, K, elem=elem, b_gain=dev_bf16(gb))
    torch.cuda.synchronize()
    g = f64(gb)
    want = oracle.mx_matmul(ac, as_, bc, bs, K, elem=elem) * g[None, :]
    mag = oracle.mx_matmul(abs_codes(ac, elem), as_, abs_codes(bc, elem), bs, K,
                           elem=elem) * np.abs(g)[None, :]
    # the gain multiply adds one float rounding (2^-24 of |H| <= sum|ab| |g|),
    # far inside the bound
    assert_close(h.cpu().numpy().astype(np.float64), want, mag, False, "gain %s" % elem)


# ------------------------------------------------------- whole backward --

def linear_bwd_pieces(gh, x, rho, gamma, w, elem, grad_x_dtype):
    """mxnorm_linear_bwd through the C entry point with a workspace of its own:
    (grad_x, grad_gamma, grad_w, pieces), pieces the intermediate operands
    where the library lays them out, each at a 256-byte boundary."""
    T, N = gh.shape
    d = x.shape[1]
    lib, e = mxnorm.load(), mxnorm.ELEMS[elem]
    half = 2 if elem == "e2m1" else 1
    gx = torch.empty(T, d, dtype=grad_x_dtype, device=DEV)
    gg, gw = torch.empty(d, device=DEV), torch.empty(N, d, device=DEV)
    ws = torch.full((lib.mxnorm_linear_bwd_workspace_bytes(T, N, d, e),), 0xA5, dtype=torch.uint8,
                    device=DEV)
    mxnorm._check(lib.mxnorm_linear_bwd(
        gh.data_ptr(), x.data_ptr(), rho.data_ptr(), mxnorm._ptr(gamma), w.data_ptr(), T, N, d, 32, e,
        mxnorm.OUT_DTYPES[grad_x_dtype], gx.data_ptr(), gg.data_ptr(), gw.data_ptr(), ws.data_ptr(),
        ws.numel(), mxnorm._stream(ws.device)))
    torch.cuda.synchronize()
    pieces, at = {}, 0
    for name, rows, cols in (("gh", T, N // half), ("gh_s", T, N // 32), ("wt", d, N // half),
                             ("wt_s", d, N // 32), ("ght", N, T // half), ("ght_s", N, T // 32),
                             ("xt", d, T // half), ("xt_s", d, T // 32), ("gz", T, 2 * d)):
        pieces[name] = ws[at:at + rows * cols].view(rows, cols)
        at += -(-rows * cols // 256) * 256
    pieces["gz"] = pieces["gz"].view(torch.bfloat16)
    return gx, gg, gw, pieces


def same_bytes(t, want, ctx):
    got = t.cpu().numpy()
    bad = np.argwhere(got != want)
    assert bad.size == 0, "%s: %d bytes differ, first %s got %#x want %#x" % (
        ctx, len(bad), bad[0], got[tuple(bad[0])], want[tuple(bad[0])])


# (T, N, d) and how the two products are computed there: in one launch of 64 x
# 128 tiles with 2 K steps each, the smallest; with 8 and 18, 6 and 10, 6 and 4
# steps (E4M3: a ring of 3 slots comes round; either product first; d and N
# beside whole tiles); or, in 8 bits, one after the other
BACKWARDS = [(256, 256, 512, "small", "small"), (1024, 2304, 768, "small", "small"),
             (768, 1280, 416, "small", "small"), (768, 512, 416, "small", "small"),
             (512, 768, 288, "apart", "small")]


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
@pytest.mark.parametrize("T,N,d,way8,way4", BACKWARDS)
def test_mxnorm_linear_backward(elem, T, N, d, way8, way4):
    from test_gpu_gemm import abs_codes, assert_close, oracle_product
    assert launch_rules.pair_plan(T, N, d, elem)[0] == (way8 if elem == "e4m3" else way4)
    rng = np.random.default_rng(17)
    xb = synth.gaussian(T, d, seed=21, scale=1.3)
    whb = synth.f32_to_bf16_bits((0.05 * rng.standard_normal((N, d))).astype(np.float32))
    ghb = synth.gaussian(T, N, seed=22, scale=0.1)
    gb = synth.f32_to_bf16_bits(rng.uniform(0.5, 1.5, d).astype(np.float32))
    x, w, gh, g = dev_bf16(xb), dev_bf16(whb), dev_bf16(ghb), dev_bf16(gb)
    _, _, rho = mxnorm.mxnorm_mx_fwd(x, block=32, elem=elem)
    gx, gg, gw, P = linear_bwd_pieces(gh, x, rho, g, w, elem, torch.float32)
    rho_np = rho.cpu().numpy()

    # the Python call is the same call: deterministic, so the same bits
    for a, b in zip((gx, gg, gw), mxnorm.mxnorm_linear_bwd(gh, x, rho, g, w, elem=elem,
                                                          grad_x_dtype=torch.float32)):
        assert torch.equal(a, b)

    # the casts, bit for bit
    hc, hs = oracle.mxcast_gain(ghb, None, B=32, elem=elem)
    wc, ws = oracle.mxcast_t(whb, None, B=32, elem=elem)
    tc, ts = oracle.mxcast_t(ghb, None, B=32, elem=elem)
    xc, xs = oracle.mxcast_t(xb, rho_np, B=32, elem=elem)
    for name, want in (("gh", hc), ("gh_s", hs), ("wt", wc), ("wt_s", ws), ("ght", tc),
                       ("ght_s", ts), ("xt", xc), ("xt_s", xs)):
        same_bytes(P[name], want, "%s %s" % (elem, name))

    # stage 1: grad_Z = MXCast(grad_H) MXCast_N(W)
    gz_o, gz_mag = oracle_product(hc, hs, wc, ws, N, elem)
    assert_close(P["gz"].float().cpu().numpy().astype(np.float64), gz_o, gz_mag, True, "grad_Z")

    # stage 2: the STE on that grad_Z
    gzb = bits_of(P["gz"])
    wx, wg = oracle.ste_bwd(xb, gzb, gb, rho_np)
    terms, gsum = ste_bounds(xb, gzb, gb, rho_np)
    assert (np.abs(gx.cpu().numpy() - wx) <= 2.0 ** -21 * terms + 2.0 ** -22 * np.abs(wx)
            + 1e-37).all()
    assert (np.abs(gg.cpu().numpy() - wg) <= 2.0 ** -16 * gsum + 1e-37).all()

    # stage 3: grad_W = (MXCast(grad_H^T) MXCast(rho~ X)^T) gamma
    gw_o, gw_mag = oracle_product(tc, ts, xc, xs, T, elem)
    gw_o, gw_mag = gw_o * f64(gb)[None, :], gw_mag * np.abs(f64(gb))[None, :]
    assert_close(gw.cpu().numpy().astype(np.float64), gw_o, gw_mag, False, "grad_W")
    if (T, N, d) != (256, 256, 512):
        return

    # and the whole thing approximates the float64 RMSNorm-linear gradient:
    # the oracle's own chain is 5.6% (E4M3) and 16.8% (E2M1) away here, from
    # the 8- or 4-bit casts and rho~'s error at d = 512 (16 blocks per row)
    xs64 = f64(xb)
    S = np.sqrt(np.mean(xs64 ** 2, axis=1, keepdims=True))
    gw_ref = f64(ghb).T @ (xs64 / S) * f64(gb)[None, :]
    rel = np.linalg.norm(gw.cpu().numpy() - gw_ref) / np.linalg.norm(gw_ref)
    assert rel < (0.10 if elem == "e4m3" else 0.30), rel


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
@pytest.mark.parametrize("T,N,d", [
    (256, 512, 256),        # one launch each in 8 bits, a shared one of small tiles in 4
    (1024, 2304, 768),      # a shared launch of small tiles, several K steps
    (4096, 6144, 4096),     # 384 and 256 tiles: both products in one launch
    (4352, 6400, 4128),     # 425 and 289 tiles, the last column of cells 32 wide
    (8192, 2560, 2080),     # 90 and 288 tiles
    (1280, 12544, 544),     # one launch each; grad_H's cast in XCD ranges, with a partial group
    (256, 256, 16), (512, 256, 48), (256, 768, 272),   # d an odd multiple of 16
])
def test_linear_backward_equals_its_parts(elem, T, N, d):
    # the one-call backward against the library's own entry points called one
    # by one.  Codes are the same bits; a product may add its K steps in
    # another grouping, which moves float sums by at most 2^-22 of sum |ab|
    # (a bf16 grad_Z then by one unit in rare elements).
    g = torch.Generator(device=DEV)
    g.manual_seed(T + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)
    x, gh, w = rnd(T, d), 0.01 * rnd(T, N), 0.02 * rnd(N, d)
    gam = 1 + 0.1 * rnd(d)
    _, _, rho = mxnorm.mxnorm_mx_fwd(x, block=16 if d % 32 else 32, elem=elem)
    gx, gg, gw = mxnorm.mxnorm_linear_bwd(gh, x, rho, gam, w, elem=elem, grad_x_dtype=torch.float32)
    a, as_ = mxnorm.mx_cast_fwd(gh, None, elem=elem)
    b, bs = mxnorm.mx_cast_t_fwd(w, None, elem=elem)
    gz = mxnorm.mx_matmul_fwd(a, as_, b, bs, N, elem=elem, out_dtype=torch.bfloat16)
    wx, wg = mxnorm.mxnorm_ste_bwd(x, gz, gam, rho, out_dtype=torch.float32)
    a, as_ = mxnorm.mx_cast_t_fwd(gh, None, elem=elem)
    b, bs = mxnorm.mx_cast_t_fwd(x, rho, elem=elem)
    ww = mxnorm.mx_matmul_fwd(a, as_, b, bs, T, elem=elem, out_dtype=torch.float32, b_gain=gam)
    torch.cuda.synchronize()
    for name, got, want in (("grad_x", gx, wx), ("grad_gamma", gg, wg), ("grad_w", gw, ww)):
        assert torch.isfinite(got).all(), name
        err = float((got - want).norm() / want.norm())
        assert err <= (1e-6 if name == "grad_w" else 1e-4), (name, err)


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
def test_linear_backward_special_values(elem):
    # zero rows and columns, subnormals, an infinity and a NaN in grad_H, zeros
    # and subnormals in W and X: the one-call backward's codes and scales are
    # the parts' bytes (the oracle's for grad_H and W), it has the parts' NaNs,
    # and their values elsewhere
    T, N, d = 512, 768, 288
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)
    x, gh, w, gam = rnd(T, d), rnd(T, N), rnd(N, d), 1 + 0.1 * rnd(d)
    gh[7], gh[:, 33] = 0, 0
    gh[64:96, 128:160] *= 2.0 ** -126
    gh[3, 5], gh[200, 700] = float("nan"), float("-inf")
    w[:, 9], w[32:64, 40:72] = 0, w[32:64, 40:72] * 2.0 ** -126
    x[64:128, 100:140] *= 2.0 ** -126
    _, _, rho = mxnorm.mxnorm_mx_fwd(x, elem=elem)
    gx, gg, gw, P = linear_bwd_pieces(gh, x, rho, gam, w, elem, torch.float32)
    a, as_ = mxnorm.mx_cast_fwd(gh, None, elem=elem)
    b, bs = mxnorm.mx_cast_t_fwd(w, None, elem=elem)
    at, at_s = mxnorm.mx_cast_t_fwd(gh, None, elem=elem)
    xt, xt_s = mxnorm.mx_cast_t_fwd(x, rho, elem=elem)
    for name, want in (("gh", a), ("gh_s", as_), ("wt", b), ("wt_s", bs), ("ght", at),
                       ("ght_s", at_s), ("xt", xt), ("xt_s", xt_s)):
        same_bytes(P[name], want.cpu().numpy(), "%s %s" % (elem, name))
    for (c, sc), (oc, os_) in (((a, as_), oracle.mxcast_gain(bits_of(gh), None, B=32, elem=elem)),
                               ((at, at_s), oracle.mxcast_t(bits_of(gh), None, B=32, elem=elem)),
                               ((b, bs), oracle.mxcast_t(bits_of(w), None, B=32, elem=elem))):
        same_bytes(c, oc, elem)
        same_bytes(sc, os_, elem)
    gz = mxnorm.mx_matmul_fwd(a, as_, b, bs, N, elem=elem, out_dtype=torch.bfloat16)
    wx, _ = mxnorm.mxnorm_ste_bwd(x, gz, gam, rho, out_dtype=torch.float32)
    a, as_ = mxnorm.mx_cast_t_fwd(gh, None, elem=elem)
    b, bs = mxnorm.mx_cast_t_fwd(x, rho, elem=elem)
    ww = mxnorm.mx_matmul_fwd(a, as_, b, bs, T, elem=elem, out_dtype=torch.float32, b_gain=gam)
    torch.cuda.synchronize()
    assert torch.isnan(gg).all()                 # rows 3 and 200 reach every column
    for name, got, want in (("grad_x", gx, wx), ("grad_w", gw, ww)):
        nan = torch.isnan(want)
        assert nan.any() and not nan.all(), name
        assert torch.equal(torch.isnan(got), nan), name
        err = float((got - want)[~nan].norm() / want[~nan].norm())
        assert err <= (1e-6 if name == "grad_w" else 1e-4), (name, err)


@pytest.mark.parametrize("elem", ["e4m3", "e2m1"])
def test_linear_backward_large_tiles_sampled(elem):
    # 425 and 289 tiles of 256 x 256 in one launch, shared out by load, the last
    # column of them 32 wide: sampled rows of grad_Z and grad_W, every column,
    # against the oracle's products of the call's own operands (which are the
    # parts' bytes)
    from test_gpu_gemm import assert_close, oracle_product, tile_sample
    T, N, d = 4352, 6400, 4128
    assert launch_rules.pair_plan(T, N, d, elem)[0] == "large"
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)
    x, gh, w, gam = rnd(T, d), 0.01 * rnd(T, N), 0.02 * rnd(N, d), 1 + 0.1 * rnd(d)
    _, _, rho = mxnorm.mxnorm_mx_fwd(x, elem=elem)
    _, _, gw, P = linear_bwd_pieces(gh, x, rho, gam, w, elem, torch.bfloat16)
    for names, cast in ((("gh", "gh_s"), mxnorm.mx_cast_fwd(gh, None, elem=elem)),
                        (("ght", "ght_s"), mxnorm.mx_cast_t_fwd(gh, None, elem=elem)),
                        (("wt", "wt_s"), mxnorm.mx_cast_t_fwd(w, None, elem=elem)),
                        (("xt", "xt_s"), mxnorm.mx_cast_t_fwd(x, rho, elem=elem))):
        for n, t in zip(names, cast):
            assert torch.equal(P[n], t), n
    H = {k: v.cpu().numpy() for k, v in P.items() if k != "gz"}
    rows = tile_sample(T, lead=2, extra=4)
    want, mag = oracle_product(H["gh"][rows], H["gh_s"][rows], H["wt"], H["wt_s"], N, elem)
    got = P["gz"][torch.from_numpy(rows).to(DEV)].float().cpu().numpy().astype(np.float64)
    assert_close(got, want, mag, True, "grad_Z %s" % elem)
    rows = tile_sample(N, lead=2, extra=4)
    want, mag = oracle_product(H["ght"][rows], H["ght_s"][rows], H["xt"], H["xt_s"], T, elem)
    f = gam.double().cpu().numpy()
    got = gw[torch.from_numpy(rows).to(DEV)].cpu().numpy().astype(np.float64)
    assert_close(got, want * f, mag * np.abs(f), False, "grad_W %s" % elem)


def test_transpose_stream_reference_moves_the_bytes():
    # the column cast's stream reference (a bandwidth denominator) really
    # reads x and rho and writes the transposed bytes it claims to
    from paper_2603_13180_amd import streamref
    R, C = 256, 512
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    x = torch.randn(R, C, generator=g, device=DEV).to(torch.bfloat16)
    rho = torch.rand(R, generator=g, device=DEV) + 0.5
    out = torch.empty(C, R, dtype=torch.uint8, device=DEV)
    small = torch.empty(C, R // 32, dtype=torch.uint8, device=DEV)
    streamref.stream_reference_transpose(x, rho, out, small)
    torch.cuda.synchronize()
    xb = x.view(torch.int16).cpu().numpy().astype(np.uint16)
    hi = (xb >> 8).astype(np.uint8)
    assert np.array_equal(out.cpu().numpy(), hi.T)
    rb = rho.cpu().numpy().view(np.uint32)
    want = (hi[0::32, :].T ^ (rb[0::32] & 0xFF)[None, :]).astype(np.uint8)
    assert np.array_equal(small.cpu().numpy(), want)
