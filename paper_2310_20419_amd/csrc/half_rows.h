// The half-precision copy of float32 rows.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave_prims.h"

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// The half-precision copy of float32 rows that the first form's Gram block is computed from: row i is h_i, the binary16
// rounding of (x_i - centre) 2^exponent, zeros up to rowbytes.  Distances do not depend on the centre, the mean of a
// sample of rows, which keeps the rounding small for rows far from the origin; the exponent puts the sample's root mean
// square near 2^-4, so that coordinates a million times larger still fit (what does not, or is not finite, becomes a NaN,
// and every pair of its row is left to the exact routine).  With r_i = |(x_i - centre) 2^exponent - h_i|, a Euclidean norm
// measured for every row in double precision, r_i <= share |h_i| + rest holds for all rows.
struct HalfPar {
    u32 share_bits, rest_bits;     // bits of non-negative floats order like the floats
    int exponent, pad;
};
struct HalfRows {
    const char *rows = nullptr;
    u32 rowbytes = 0;
    const HalfPar *par = nullptr;
};
#define HALF_SAMPLE 512          // rows the centre is the mean of
