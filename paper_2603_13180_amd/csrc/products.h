// products.h -- what the composed MXNormLinear calls use of the entry points'
// implementation (internal; not part of the C ABI): the entry points' argument
// checks, which launch nothing, and the parts of the backward that share a
// launch, whose arguments the caller has checked.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mxnorm.h"

namespace mxk {

// mxnorm_mx_fwd's and mx_cast_fwd's checks; coef <= 0 becomes the table's.
mx_status check_mxnorm(const void *x, int64_t T, int64_t d, int block, int elem, int p, float &coef,
                       float eps, int scale_mode, const uint8_t *codes, const uint8_t *scales,
                       const float *rho);
mx_status check_cast(const void *x, const void *gamma, int64_t T, int64_t d, int block, int elem,
                     int scale_mode, const uint8_t *codes, const uint8_t *scales);

} // namespace mxk

namespace mxg {

// out = dec(a) dec(b)^T (times gain per column), as mx_matmul_fwd's arguments;
// M, N > 0.
struct Product {
    const uint8_t *a, *as, *b, *bs;
    int64_t M, N, K;
    const void *gain;
    void *out;
};

// mx_matmul_fwd's checks.
mx_status check_product(const Product &P, int block, int elem, int out_dtype);

// A product with float output and one with bf16 output that do not depend on
// each other, on one stream: within mx_matmul_fwd's bound, in one launch or
// two, so the sums may be taken in another order than by two mx_matmul_fwd calls.
mx_status matmul_pair(const Product &f32, const Product &bf16, int elem, hipStream_t stream);

} // namespace mxg

namespace mxb {

// mx_cast_t_fwd's and mxnorm_ste_bwd's checks.
mx_status check_cast_t(const void *x, const float *rho, int64_t R, int64_t C, int block, int elem,
                       int scale_mode, const uint8_t *codes, const uint8_t *scales);
mx_status check_ste(const void *x, const void *grad_z, const void *gamma, const float *rho,
                    int64_t T, int64_t d, int out_dtype, const void *grad_x, const float *grad_gamma,
                    const void *workspace, size_t workspace_bytes);

// Codes and scales of the backward's casts, laid out as the entry points of
// the single casts do (RCEIL, blocks of 32).
struct BackwardCasts {
    uint8_t *gh, *gh_s;   // grad_H [T, N] along N
    uint8_t *ght, *ght_s; // grad_H^T [N, T] along T
    uint8_t *wt, *wt_s;   // W^T [d, N] along N
    uint8_t *xt, *xt_s;   // (rho X)^T [d, T] along T
};

// T and N multiples of 128, d of 16; grad_h, x, w 16-byte aligned.
mx_status backward_casts(const void *grad_h, const void *x, const float *rho, const void *w,
                         int64_t T, int64_t N, int64_t d, int elem, const BackwardCasts &o,
                         hipStream_t stream);

} // namespace mxb
