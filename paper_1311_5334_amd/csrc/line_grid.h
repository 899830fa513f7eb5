// line_grid.h -- geometry of the grids the counting kernel walks: how large
// cells and slabs are, which cells list a grain, and where a line crosses a
// slab's plane. Plain arithmetic, so that the host tests compile it alone.
//
// A line's class is the axis a of its largest |d| (its face) and which of sub x
// sub bins its slopes d_u / d_a, d_v / d_a in [-1, 1] fall in (u, v the other
// two axes). For each class the view is cut along a into slabs of w units, and
// each slab's middle plane into c x c cells. A line of the class crosses the
// middle plane of slab k at one point, so it looks at one cell a slab; that
// cell lists every grain of the slab that any line of the class through the
// cell can have within r. A grain h units off the middle plane is met by lines
// that cross the plane within delta |h| + r sqrt(1 + s^2) of (u - s0 h,
// v - t0 h), (s0, t0) the bin's middle slopes, delta = 1 / sub the bin's half
// width and s the largest |slope| of the bin: the grain is listed in every cell
// of that rectangle, widened by the grid's margin against the error of the
// crossing points (line_error). The exact test decides the grains.
#ifndef EMT_LINE_GRID_H
#define EMT_LINE_GRID_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace emt {

constexpr int kSubMax = 4;                           // most slope bins an axis
constexpr int kLineClasses = 3 * kSubMax * kSubMax;  // most line classes a view has
constexpr int kLineEdge = 2048;                // cells of a plane along u or v
constexpr int kLineMargin = 4;                 // least margin of a rectangle (units)
constexpr int kPackSpan = 2048;                // units a packed word's u and v reach either way
// fractional bits of a crossing point: its cell is the upper half word
constexpr int kLineBits = 16;
constexpr float kLineOne = (float)(1 << kLineBits);
static_assert((unsigned long long)kLineEdge << kLineBits <= 1ull << 31, "crossing points");
// Records a view may use per grain, when tables hold nc classes.
__host__ __device__ inline uint32_t line_recs(int nc) { return (uint32_t)(nc + nc / 4); }
constexpr uint32_t kLineEnt = 12;              // list words of a class per grain

// Per view: the grids the counting kernel walks, written by k_grid. Face a
// holds sub * sub classes of ns[a] planes each.
struct LineGrid {
    int32_t sub;           // slope bins an axis (0: no lines)
    int32_t c, w;          // cell edge and slab thickness (units)
    int32_t margin;        // a rectangle's widening (units)
    int32_t reach;         // cells start this far below the bounding box
    float ic;              // 1 / c
    int32_t packed;        // list words hold the grains' coordinates
    int32_t ns[3];         // slabs along the face's axis
    int32_t nu[3], nv[3];  // cells of a plane
    int32_t bu[3];         // records (8 x 4 cells each) in a row of records
    uint32_t plane[3];     // records from one plane to the next
    uint32_t face_off[3];  // the face's first record, from the view's first
};

__host__ __device__ inline int line_u(int a) { return a == 0 ? 1 : 0; }
__host__ __device__ inline int line_v(int a) { return a == 2 ? 1 : 2; }

// Largest distance, in a plane's u or v, between a grain and the cells that
// list it.
__host__ __device__ inline int line_reach(int w, int r, int margin) {
    return w / 2 + 1 + (int)(1.42f * (float)r) + margin + 1;
}

// Most units a crossing point and a rectangle's edge are off together: below 1
// from FP32 (coordinates up to 2^18), up to a fixed-point step where the
// line's first crossing is cut, and half a step for each slab from there.
__host__ __device__ inline int line_error(double c, double w, long long span) {
    return 1 + (int)ceil(c * (1.0 / (1 << kLineBits)) * (1.0 + 0.5 * (double)span / w));
}

// c and w grow until the view's records fit their share; c is at least
// `spread` times the half side of a grain's largest rectangle, and no more than
// 3/4 w, which keeps the crossing points exact enough for the least margin, or
// 3/2 w where a rectangle is that wide itself (one bin and spread 2: 2 half >
// w). It ends: as spread / (2 sub) is below that limit, a larger w meets it; and
// once w passes the span, the planes are one slab and at most 5 x 5 cells, two
// records, as c >= w / 4, and two grains' share holds those.
__host__ __device__ inline LineGrid line_grid(uint32_t n, const long long *span, const int *tab,
                                              int nc, int r, double spread) {
    LineGrid L = {};
    if (n < 2) return L;
    int sub = tab[2];
    while (3 * sub * sub > nc) --sub;
    L.sub = sub;
    const unsigned long long cap = (unsigned long long)line_recs(nc) * n;
    long long most = span[0] > span[1] ? span[0] : span[1];
    most = span[2] > most ? span[2] : most;
    const double limit = spread < 1.5 * sub ? 0.75 : 1.5;
    // (crossing points are then below 2^31 / kLineOne cells)
    double w = tab[1] > 64 ? tab[1] : 64;
    double c = fmax(fmax((double)tab[0], 0.25 * w), 32.0);
    for (;;) {
        const int err = line_error(c, w, most);
        L.margin = err > kLineMargin ? err : kLineMargin;
        const double need = (0.5 * w / sub + 1.4143 * r + L.margin) * spread + 2.0;
        if (c < need) {
            c = need;
            continue;
        }
        if (c > limit * w) {
            w *= 1.19;
            continue;
        }
        L.c = (int)c;
        L.w = (int)w;
        L.reach = line_reach(L.w, r, L.margin);
        unsigned long long off = 0;
        bool ok = true;
        for (int a = 0; a < 3; ++a) {
            const long long ns = span[a] / L.w + 1;
            const long long nu = (span[line_u(a)] + 2 * L.reach) / L.c + 1;
            const long long nv = (span[line_v(a)] + 2 * L.reach) / L.c + 1;
            ok = ok && ns <= 65535 && nu <= kLineEdge && nv <= kLineEdge;
            L.ns[a] = (int)ns;
            L.nu[a] = (int)nu;
            L.nv[a] = (int)nv;
            L.bu[a] = (int)((nu + 7) / 8);
            L.plane[a] = (uint32_t)(L.bu[a] * ((nv + 3) / 4));
            L.face_off[a] = (uint32_t)off;
            off += (unsigned long long)L.plane[a] * ns * (sub * sub);
        }
        if (ok && off <= cap) break;
        c *= 1.19;
        w *= 1.19;
    }
    L.ic = 1.0f / (float)L.c;
    L.packed = 8 * L.c < kPackSpan && 2 * L.reach < kPackSpan ? 1 : 0;
    return L;
}

// Half side of the rectangle, at h = 0, of a class with largest |slope| s.
__host__ __device__ inline float line_half(int r, float s, int margin) {
    return (float)r * sqrtf(1.0f + s * s) + (float)margin;
}

// Cells j0 .. j1 of [lo, hi] along u (or v) that list a grain at x there, h off
// its slab's middle plane; s0, delta: the bin's middle slope and half width,
// half: line_half.
__host__ __device__ inline void line_cells(const LineGrid &L, float x, float h, float s0,
                                           float delta, float half, int lo, int hi, int &j0,
                                           int &j1) {
    const float side = fmaf(delta, fabsf(h), half);
    const float at = x + (float)L.reach - s0 * h;
    const int a = (int)((at - side) * L.ic), b = (int)((at + side) * L.ic);
    j0 = a > lo ? a : lo;
    j1 = b < hi ? b : hi;
}

// Where a line through (ga, x) of slope s crosses slab 0's plane along u (or
// v), in cells, and how far on it crosses the next slab's.
struct LineCross {
    float x0, step;
    __host__ __device__ int fixed0() const { return (int)(x0 * kLineOne); }
    __host__ __device__ int fixed_step() const { return (int)rintf(step * kLineOne); }
};
__host__ __device__ inline LineCross line_cross(const LineGrid &L, float s, float ga, int x) {
    const float w = (float)L.w;
    return {fmaf(s, 0.5f * w - ga, (float)(x + L.reach)) * L.ic, s * w * L.ic};
}

}  // namespace emt

#endif
