// Host-only check of seed_rows.h: the layer of every row of the largest boxes,
// with a reciprocal an ulp off either way.
#include <algorithm>
#include <cmath>
#include <cstdio>

#include "seed_rows.h"

using namespace emt;

int main() {
    int failures = 0;
    const long long most = (1ll << 22) + 4096;  // cells of a view
    for (int ny = 1; ny <= 8193; ny += ny < 300 ? 1 : 7)
        for (int ulp = -1; ulp <= 1; ++ulp) {
            float rcp = 1.0f / (float)ny;
            if (ulp) rcp = std::nextafterf(rcp, ulp > 0 ? 1e30f : 0.0f);
            const float inv = rcp * kRowsMore;
            const long long layers = std::min(8193ll, most / ny);
            for (long long z = 0; z < layers; ++z)
                for (long long y : {0ll, 1ll, ny / 2ll, ny - 2ll, ny - 1ll}) {
                    if (y < 0 || y >= ny) continue;
                    const int got = row_layer((int)(z * ny + y), ny, inv);
                    if (got != z && failures++ < 5)
                        std::printf("FAIL row %lld of %d a layer: layer %d, not %lld\n", z * ny + y,
                                    ny, got, z);
                }
        }
    if (failures == 0) std::printf("seed rows ok\n");
    return failures ? 1 : 0;
}
