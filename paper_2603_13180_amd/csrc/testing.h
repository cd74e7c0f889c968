// testing.h -- what the library's own tests ask of its launch rules.  Exported
// by libmxnorm.so but not part of the C ABI: names and arguments may change.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mxnorm.h"

extern "C" {

// Lanes per row the norm/cast entry points launch for [T, d]; 0 if none fits.
// kind: 0 RMSNorm, 1 MXNorm, 2 plain cast, 3 post-round MXNorm; fmt: 0..2
// MXFP8 with blocks of 16, 32, 64, 3..5 MXFP4, 6 NVFP4; gain: a gamma is given.
int mxt_norm_team(int64_t T, int64_t d, int kind, int fmt, int gain);

// Tile shapes of mxt_product_plan: 0 .. 6 = 16 x 32, 32 x 32, 32 x 64 and 64 x
// 64 with K split over the waves, 64 x 128 and 128 x 128 rings, 256 x 256.
//
// How mx_matmul_fwd computes [M, K] x [N, K]^T on `units` compute units:
// returns the tile shape, or -1 for sizes it refuses; *whole > 0: that many
// cells of 256 x 256 in a first launch and the rest in tiles of *tail in a
// second.  *us: the estimate the choice was made by.
int mxt_product_plan(int64_t M, int64_t N, int64_t K, int elem, int units, int *whole, int *tail,
                     double *us);

// How mxnorm_linear_bwd computes its two products (0: float output, 1: bf16):
// 0 one after the other, 1 in one launch of 256 x 256 tiles, 2 in one launch
// of 64 x 128 tiles; -1: refused.  us[3]: the three estimates.
int mxt_pair_plan(int64_t M0, int64_t N0, int64_t K0, int64_t M1, int64_t N1, int64_t K1, int elem,
                  int units, double *us);

// mx_matmul_fwd with blocks of 32 in a given way, so that every kernel is
// reached at sizes the oracle can check: in tiles of `shape`, or, whole > 0,
// that many cells of 256 x 256 in a first launch and the rest in tiles of
// `shape`; the persistent kernels as on `units` compute units (0: the
// device's, which is also the most), so that a workgroup takes many tiles.
// Same argument checks as mx_matmul_fwd.
mx_status mxt_matmul(const uint8_t *a_codes, const uint8_t *a_scales, const uint8_t *b_codes,
                     const uint8_t *b_scales, int64_t M, int64_t N, int64_t K, int elem,
                     const void *b_gain, int out_dtype, void *out, int shape, int whole, int units,
                     hipStream_t stream);

// One product of mxt_matmul_pair, as the arguments of mx_matmul_fwd.
typedef struct MxtProduct {
    const uint8_t *a, *as, *b, *bs;
    int64_t M, N, K;
    const void *gain;
    void *out;
} MxtProduct;

// Two products as mxnorm_linear_bwd computes them, one with float and one with
// bf16 output, in a given way (mxt_pair_plan's numbers).  MX_EINVAL if the
// large tiles cannot be shared out.
mx_status mxt_matmul_pair(const MxtProduct *f32, const MxtProduct *bf16, int elem, int mode,
                          int units, hipStream_t stream);

} // extern "C"
