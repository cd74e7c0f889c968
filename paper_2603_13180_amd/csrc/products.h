// products.h -- two MX products launched together (internal; not part of the
// C ABI).
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
