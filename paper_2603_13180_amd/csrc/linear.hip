// linear.hip -- the MXNormLinear forward and backward as one call each
// (Sec. 3.7; the implementation appendix's mx_norm_linear_forward and
// mx_norm_linear_backward): the norm, cast, product and straight-through-
// estimator kernels of this library, launched one after the other on the
// caller's stream, their intermediate operands in the caller's workspace.
//
// At small sizes these calls are bound by the host: from Python, eight
// entry-point calls and a dozen output allocations took 93 us for a 1024 x
// 768 x 2304 backward whose kernels take 70.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "mxnorm.h"
#include "products.h"
#include "status.h"

namespace {

// Pieces of a workspace, each at a 256-byte boundary.
struct Carver {
    uint8_t *base;
    size_t used = 0;
    uint8_t *take(size_t bytes)
    {
        uint8_t *p = base ? base + used : nullptr;
        used += (bytes + 255) & ~(size_t)255;
        return p;
    }
};

size_t code_bytes(int64_t rows, int64_t cols, int elem)
{
    return (size_t)rows * (size_t)cols / (elem == MX_ELEM_E2M1 ? 2 : 1);
}

struct FwdSpace {
    uint8_t *codes, *scales;
    size_t bytes;
    FwdSpace(void *ws, int64_t T, int64_t d, int block, int elem)
    {
        Carver c{static_cast<uint8_t *>(ws)};
        codes = c.take(code_bytes(T, d, elem));
        scales = c.take((size_t)T * (size_t)(d / block));
        bytes = c.used;
    }
};

struct BwdSpace {
    uint8_t *gh, *gh_s, *wt, *wt_s, *ght, *ght_s, *xt, *xt_s, *gz, *ste;
    size_t ste_bytes, bytes;
    BwdSpace(void *ws, int64_t T, int64_t N, int64_t d, int elem)
    {
        Carver c{static_cast<uint8_t *>(ws)};
        gh = c.take(code_bytes(T, N, elem));
        gh_s = c.take((size_t)T * (size_t)(N / 32));
        wt = c.take(code_bytes(d, N, elem));
        wt_s = c.take((size_t)d * (size_t)(N / 32));
        ght = c.take(code_bytes(N, T, elem));
        ght_s = c.take((size_t)N * (size_t)(T / 32));
        xt = c.take(code_bytes(d, T, elem));
        xt_s = c.take((size_t)d * (size_t)(T / 32));
        gz = c.take((size_t)T * (size_t)d * 2);
        ste_bytes = mxnorm_ste_bwd_workspace_bytes(T, d);
        ste = c.take(ste_bytes);
        bytes = c.used;
    }
};

bool known(int elem) { return elem == MX_ELEM_E4M3 || elem == MX_ELEM_E2M1; }

mx_status check_workspace(const void *ws, size_t have, size_t need)
{
    if (need > 0 && (!ws || ((uintptr_t)ws & 255) != 0 || have < need))
        return mxk::fail(MX_EINVAL, "a 256-byte aligned workspace of %zu bytes is needed", need);
    return MX_OK;
}

} // namespace

extern "C" {

size_t mxnorm_linear_fwd_workspace_bytes(int64_t T, int64_t d, int block, int elem)
{
    if (T <= 0 || d <= 0 || block <= 0 || !known(elem))
        return 0;
    return FwdSpace(nullptr, T, d, block, elem).bytes;
}

mx_status mxnorm_linear_fwd(const void *x, int64_t T, int64_t d, const uint8_t *w_codes,
                            const uint8_t *w_scales, int64_t N, int block, int elem, int p,
                            float coef, float eps, int scale_mode, int out_dtype, void *out,
                            float *rho, void *workspace, size_t workspace_bytes,
                            hipStream_t stream)
{
    mxk::clear_error();
    mx_status st = check_workspace(workspace, workspace_bytes,
                                   mxnorm_linear_fwd_workspace_bytes(T, d, block, elem));
    if (st != MX_OK)
        return st;
    const FwdSpace s(workspace, T, d, block > 0 ? block : 1, elem);
    // both parts' checks come before the first launch
    float c = coef;
    if ((st = mxk::check_mxnorm(x, T, d, block, elem, p, c, eps, scale_mode, s.codes, s.scales,
                                rho)) != MX_OK ||
        (st = mxg::check_product({s.codes, s.scales, w_codes, w_scales, T, N, d, nullptr, out},
                                 block, elem, out_dtype)) != MX_OK ||
        (st = mxnorm_mx_fwd(x, T, d, block, elem, p, coef, eps, scale_mode, s.codes, s.scales, rho,
                            stream)) != MX_OK)
        return st;
    return mx_matmul_fwd(s.codes, s.scales, w_codes, w_scales, T, N, d, block, elem, nullptr,
                         out_dtype, out, stream);
}

size_t mxnorm_linear_bwd_workspace_bytes(int64_t T, int64_t N, int64_t d, int elem)
{
    if (T <= 0 || N <= 0 || d <= 0 || !known(elem))
        return 0;
    return BwdSpace(nullptr, T, N, d, elem).bytes;
}

mx_status mxnorm_linear_bwd(const void *grad_h, const void *x, const float *rho,
                            const void *gamma, const void *w, int64_t T, int64_t N, int64_t d,
                            int block, int elem, int out_dtype, void *grad_x, float *grad_gamma,
                            float *grad_w, void *workspace, size_t workspace_bytes,
                            hipStream_t stream)
{
    mxk::clear_error();
    mx_status st = check_workspace(workspace, workspace_bytes,
                                   mxnorm_linear_bwd_workspace_bytes(T, N, d, elem));
    if (st != MX_OK)
        return st;
    const BwdSpace s(workspace, T, N, d, elem);
    const int mode = MX_SCALE_RCEIL;
    const mxg::Product gz{s.gh, s.gh_s, s.wt, s.wt_s, T, d, N, nullptr, s.gz};
    const mxg::Product gw{s.ght, s.ght_s, s.xt, s.xt_s, N, d, T, gamma, grad_w};
    // the parts' checks, in the parts' order, before the first launch
    if ((st = mxk::check_cast(grad_h, nullptr, T, N, block, elem, mode, s.gh, s.gh_s)) != MX_OK ||
        (st = mxb::check_cast_t(w, nullptr, N, d, block, elem, mode, s.wt, s.wt_s)) != MX_OK ||
        (st = mxg::check_product(gz, block, elem, MX_OUT_BF16)) != MX_OK ||
        (st = mxb::check_ste(x, s.gz, gamma, rho, T, d, out_dtype, grad_x, grad_gamma, s.ste,
                             s.ste_bytes)) != MX_OK ||
        (st = mxb::check_cast_t(grad_h, nullptr, T, N, block, elem, mode, s.ght, s.ght_s)) != MX_OK ||
        (st = mxb::check_cast_t(x, rho, T, d, block, elem, mode, s.xt, s.xt_s)) != MX_OK ||
        (st = mxg::check_product(gw, block, elem, MX_OUT_F32)) != MX_OK)
        return st;
    // (T, N and d are positive here: a product's K, a cast's columns)
    // grad_Z = MXCast(grad_H) MXCast_N(W), both blocked along N; grad_W =
    // (MXCast(grad_H^T) MXCast(rho~ X)^T) . gamma, blocked along T; then
    // grad_X and grad_gamma
    if ((st = mxb::backward_casts(grad_h, x, rho, w, T, N, d, elem,
                                  {s.gh, s.gh_s, s.ght, s.ght_s, s.wt, s.wt_s, s.xt, s.xt_s},
                                  stream)) != MX_OK ||
        (st = mxg::matmul_pair(gw, gz, elem, stream)) != MX_OK)
        return st;
    return mxnorm_ste_bwd(x, s.gz, gamma, rho, T, d, out_dtype, grad_x, grad_gamma, s.ste,
                          s.ste_bytes, stream);
}

} // extern "C"
