// seed_rows.h -- the rows of a seed's box of cells, numbered along y, then z.
// Plain arithmetic, so that the host tests compile it alone.
#ifndef EMT_SEED_ROWS_H
#define EMT_SEED_ROWS_H

#include <hip/hip_runtime.h>

namespace emt {

// What a quotient rounded by a reciprocal is widened by, so that it is never
// below the exact one: more than an ulp of the reciprocal and of the product.
constexpr float kRowsMore = 1.0f + 0x1p-20f;

// The z layer of row rr: rr / ny, with inv = kRowsMore / ny as an approximate
// reciprocal gives it. The product is at most 2^-19 of itself too large; there
// are at most 2^22 + 4096 cells in a view, and so rows, and 2^13 layers: it is
// one too high at most, which happens from about 800 thousand rows on.
__host__ __device__ inline int row_layer(int rr, int ny, float inv) {
    const int z = (int)((float)rr * inv);
    return z * ny > rr ? z - 1 : z;
}

}  // namespace emt

#endif
