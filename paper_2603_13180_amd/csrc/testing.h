// testing.h -- what the library's own tests ask of its launch rules.  Exported
// by libmxnorm.so but not part of the C ABI: names and arguments may change.
#pragma once

#include <stdint.h>

#include "mxnorm.h"

extern "C" {

// Lanes per row the norm/cast entry points launch for [T, d]; 0 if none fits.
// kind: 0 RMSNorm, 1 MXNorm, 2 plain cast, 3 post-round MXNorm; fmt: 0..2
// MXFP8 with blocks of 16, 32, 64, 3..5 MXFP4, 6 NVFP4; gain: a gamma is given.
int mxt_norm_team(int64_t T, int64_t d, int kind, int fmt, int gain);

} // extern "C"
