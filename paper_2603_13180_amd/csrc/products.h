// products.h -- parts of the MXNormLinear backward that share a launch
// (internal; not part of the C ABI).  Arguments are checked by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mxnorm.h"

namespace mxg {

// out = dec(a) dec(b)^T (times gain per column), as mx_matmul_fwd's arguments;
// M, N > 0.
struct Product {
    const uint8_t *a, *as, *b, *bs;
    int64_t M, N, K;
    const void *gain;
    void *out;
};

// A product with float output and one with bf16 output that do not depend on
// each other, on one stream.  Values as two mx_matmul_fwd calls.
mx_status matmul_pair(const Product &f32, const Product &bf16, int elem, hipStream_t stream);

} // namespace mxg

namespace mxb {

// Codes and scales of the backward's casts, laid out as the entry points of
// the single casts do (RCEIL, blocks of 32).
struct BackwardCasts {
    uint8_t *gh, *gh_s;   // grad_H [T, N] along N
    uint8_t *ght, *ght_s; // grad_H^T [N, T] along T
    uint8_t *wt, *wt_s;   // W^T [d, N] along N
    uint8_t *xt, *xt_s;   // (rho X)^T [d, T] along T
};

// T and N multiples of 128, d of 32; grad_h, x, w 16-byte aligned.
mx_status backward_casts(const void *grad_h, const void *x, const float *rho, const void *w,
                         int64_t T, int64_t N, int64_t d, int elem, const BackwardCasts &o,
                         hipStream_t stream);

} // namespace mxb
