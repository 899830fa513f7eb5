// Host-only check of line_grid.h: for every number of line classes, radius,
// span and density the grids exist, fit their share and hold what the kernels
// assume, and a line looks at a cell that lists every grain within r of it.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "line_grid.h"

using namespace emt;

static int failures = 0;

#define CHECK(cond, ...)                                     \
    do {                                                     \
        if (!(cond)) {                                       \
            if (failures++ < 10) {                           \
                std::printf("FAIL %s: ", #cond);             \
                std::printf(__VA_ARGS__);                    \
                std::printf("\n");                           \
            }                                                \
        }                                                    \
    } while (0)

struct Setup {
    uint32_t n;
    long long span[3];
    int tab[3], nc, r;
    double spread;
};

static void geometry(const Setup &S, const LineGrid &L) {
#define AT "n %u span %lld %lld %lld tab %d %d %d nc %d r %d spread %.2f: c %d w %d margin %d", \
        S.n, S.span[0], S.span[1], S.span[2], S.tab[0], S.tab[1], S.tab[2], S.nc, S.r, S.spread, \
        L.c, L.w, L.margin
    CHECK(L.sub >= 1 && L.sub <= S.tab[2] && 3 * L.sub * L.sub <= S.nc, AT);
    CHECK(L.c >= 32 && L.w >= 64 && L.c < 1 << 20 && L.w < 1 << 20, AT);
    CHECK(L.margin >= kLineMargin && L.reach > 0 && L.reach < 1 << 20, AT);
    const long long most = std::max(S.span[0], std::max(S.span[1], S.span[2]));
    CHECK(L.margin >= line_error(L.c, L.w + 1, most), AT);
    const double half = 0.5 * L.w / L.sub + 1.4143 * S.r + L.margin;
    CHECK(L.c + 1 >= half * S.spread, AT);
    unsigned long long off = 0;
    for (int a = 0; a < 3; ++a) {
        CHECK(L.face_off[a] == off, AT);
        CHECK(L.ns[a] >= 1 && L.ns[a] <= 65535 && (long long)L.ns[a] * L.w > S.span[a], AT);
        CHECK(L.nu[a] >= 1 && L.nu[a] <= kLineEdge && L.nv[a] >= 1 && L.nv[a] <= kLineEdge, AT);
        CHECK((long long)L.nu[a] * L.c > S.span[line_u(a)] + 2 * L.reach, AT);
        CHECK((long long)L.nv[a] * L.c > S.span[line_v(a)] + 2 * L.reach, AT);
        off += (unsigned long long)L.plane[a] * L.ns[a] * (L.sub * L.sub);
    }
    CHECK(off <= (unsigned long long)line_recs(S.nc) * S.n, AT);
    CHECK(!L.packed || (8 * L.c < kPackSpan && 2 * L.reach < kPackSpan), AT);
    // first crossing points as fixed point stay in 32 bits
    CHECK((2.0 * most + L.reach + 0.5 * L.w) / L.c * kLineOne < 2147483647.0, AT);
}

static int bin_of(float slope, int sub) {
    const int b = (int)((slope + 1.0f) * (0.5f * (float)sub));
    return b < 0 ? 0 : b > sub - 1 ? sub - 1 : b;
}

// One line through two grains of the view: its crossing points are no further
// off than the margin, and a grain near it, if it is within r, is listed by the
// cell that the line looks at in the grain's slab. Slopes by a reciprocal an ulp
// off, as the device's may be.
static unsigned long long looked = 0, hits = 0;

static void look(const Setup &S, const LineGrid &L, std::mt19937 &rng, bool edges) {
    auto pick = [&](long long lo, long long hi) {
        return lo + (long long)(rng() % (unsigned long long)(hi - lo + 1));
    };
    long long g[3], d[3];
    for (int m = 0; m < 3; ++m) g[m] = pick(0, S.span[m]);
    for (int m = 0; m < 3; ++m) d[m] = pick(-4095, 4095) / (1 + (long long)(rng() % 40));
    if (edges) {  // slopes of exactly +-1 and at bins' edges
        const int a = (int)(rng() % 3);
        const long long s = pick(1, 1000);
        for (int m = 0; m < 3; ++m) d[m] = (m == a ? 4 : pick(-4, 4)) * s;
    }
    long long ad[3];
    for (int m = 0; m < 3; ++m) ad[m] = std::llabs(d[m]);
    const int a = ad[0] >= ad[1] && ad[0] >= ad[2] ? 0 : ad[1] >= ad[2] ? 1 : 2;
    if (ad[a] == 0) return;
    const int u = line_u(a), v = line_v(a);
    float ida = 1.0f / (float)d[a];
    ida = nextafterf(ida, rng() % 2 ? 1e30f : -1e30f);
    const float slope[2] = {(float)d[u] * ida, (float)d[v] * ida};
    const int axis[2] = {u, v}, n[2] = {L.nu[a], L.nv[a]};
    // a grain beside the line, in a slab the line crosses inside the view
    long long k[3];
    k[a] = pick(0, S.span[a]);
    if (edges && rng() % 2) k[a] = k[a] / L.w * L.w;  // the slab's edge
    const int slab = (int)(k[a] / L.w);
    const double mid = (double)slab * L.w + 0.5 * L.w;
    bool near = true;
    for (int i = 0; i < 2; ++i) {
        const int m = axis[i];
        const double s = (double)d[m] / d[a], side = S.r * sqrt(1.0 + s * s);
        k[m] = std::llround((double)g[m] + (k[a] - g[a]) * s +
                            side * ((double)pick(-1000, 1000) / 1000.0));
        near = near && k[m] >= 0 && k[m] <= S.span[m];
        const double x = (double)g[m] + (mid - g[a]) * s + L.reach;
        if (x < 0.0 || x >= (double)n[i] * L.c) {
            near = false;
            continue;
        }
        ++looked;
        const LineCross X = line_cross(L, slope[i], (float)g[a], (int)g[m]);
        const double got = ((double)X.fixed0() + (double)slab * X.fixed_step()) / kLineOne * L.c;
        CHECK(fabs(got - x) <= L.margin, "sub %d c %d w %d r %d slab %d of %d: %.2f off, margin %d",
              L.sub, L.c, L.w, S.r, slab, L.ns[a], got - x, L.margin);
    }
    if (!near) return;
    __int128 sum = 0, D = 0;
    for (int m = 0; m < 3; ++m) {
        const int p = (m + 1) % 3, q = (m + 2) % 3;
        const __int128 e = (__int128)(k[p] - g[p]) * d[q] - (__int128)(k[q] - g[q]) * d[p];
        sum += e * e;
        D += (__int128)d[m] * d[m];
    }
    if (sum > (__int128)S.r * S.r * D) return;
    ++hits;
    const float delta = 1.0f / (float)L.sub, h = (float)k[a] - (float)mid;
    for (int i = 0; i < 2; ++i) {
        const float s0 = (float)(2 * bin_of(slope[i], L.sub) + 1) * delta - 1.0f;
        const float half = line_half(S.r, fabsf(s0) + delta, L.margin);
        int j0, j1;
        line_cells(L, (float)k[axis[i]], h, s0, delta, half, 0, n[i] - 1, j0, j1);
        const LineCross X = line_cross(L, slope[i], (float)g[a], (int)g[axis[i]]);
        const uint32_t at = (uint32_t)X.fixed0() + (uint32_t)slab * (uint32_t)X.fixed_step();
        const int cell = (int)(at >> kLineBits);
        CHECK(at < (uint32_t)n[i] << kLineBits && j0 <= cell && cell <= j1,
              "sub %d c %d w %d r %d slab %d of %d: cell %d of %d, listed in %d..%d (slope %.9g)",
              L.sub, L.c, L.w, S.r, slab, L.ns[a], cell, n[i], j0, j1, slope[i]);
        // the coarser grid's rectangles are of two cells at most, and words
        // that hold the coordinates hold them relative to the record's cells
        CHECK(S.spread < 2.0 || j1 - j0 <= 1, "sub %d c %d w %d r %d: cells %d..%d", L.sub, L.c,
              L.w, S.r, j0, j1);
        if (L.packed)
            for (int j : {j0, j1}) {
                const long long rel = k[axis[i]] - (j / 8) * 8ll * L.c;
                CHECK(rel >= -2048 && rel < 2048, "c %d reach %d: %lld", L.c, L.reach, rel);
            }
    }
}

int main() {
    const int tabs[][3] = {{250, 1000, 2}, {250, 800, 2}, {200, 600, 3}, {130, 500, 4},
                           {110, 400, 4}, {100, 250, 4}, {250, 800, 1}, {1, 1, 4}, {1, 1, 1},
                           {1, 1 << 18, 4}, {1 << 18, 1, 2}, {1 << 18, 1 << 18, 1}, {10, 1000, 1}};
    const long long spans[][3] = {{0, 0, 0}, {1, 0, 0}, {20000, 20000, 5000}, {28200, 28200, 0},
                                  {1 << 18, 1 << 18, 1 << 18}, {1 << 18, 300, 5000},
                                  {0, 0, 1 << 18}, {35000, 35000, 4800}};
    std::mt19937 rng(7);
    for (const auto &tab : tabs)
        for (const auto &sp : spans)
            for (int nc : {3, 12, 48})
                for (int r : {0, 1, 50, 300, 1500, 4095})
                    for (double spread : {2.0 / 3.0, 2.0})
                        for (uint32_t n : {0u, 1u, 2u, 3u, 40u, 9026u, 60000u, (1u << 20) - 1u}) {
                            Setup S{n, {sp[0], sp[1], sp[2]}, {tab[0], tab[1], tab[2]}, nc, r, spread};
                            const LineGrid L = line_grid(n, S.span, S.tab, nc, r, spread);
                            if (n < 2) {
                                CHECK(L.sub == 0, "n %u", n);
                                continue;
                            }
                            geometry(S, L);
                            for (int t = 0; t < 200; ++t) look(S, L, rng, t % 2);
                        }
    CHECK(looked > 1000000 && hits > 200000, "%llu looked at, %llu hits", looked, hits);
    if (failures == 0) std::printf("line grid ok\n");
    return failures ? 1 : 0;
}
