// deal.h -- how the counting kernel's items (seeds, or candidates when their
// members are listed) are dealt to its workgroups. Plain arithmetic, so that
// the host tests compile it alone.
//
// The items are cut into chunks of consecutive ones and workgroup b runs on
// XCD b % 8. Chunks are dealt to the XCDs in turn (as workgroups are), or
// `apart`: each XCD has an eighth of the list. Workgroup b starts with chunk
// b / 8 of its XCD's share, if the share has that many, without a counter; the
// chunks behind those are handed out by a counter an XCD.
#ifndef EMT_DEAL_H
#define EMT_DEAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace emt {

constexpr uint32_t kXcds = 8;

struct Deal {
    uint32_t n_items, size, n_chunks;  // items, items a chunk, chunks
    uint32_t per;                      // chunks of an XCD's eighth (apart)
    bool apart;
};

// Chunks of a grid of `grid` workgroups of `waves` waves that take `step`
// items at a time: one a workgroup where its waves take no more than two times
// each, else about eight, at least a time for every wave and at most `most`
// items.
__host__ __device__ inline Deal make_deal(uint32_t n_items, uint32_t step, uint32_t waves,
                                          uint32_t grid, uint32_t most, bool apart) {
    Deal D;
    const uint32_t share = n_items / grid + 1u, round = step * waves;
    if (share <= 2u * round) {
        D.size = (share + step - 1u) / step * step;
    } else {
        D.size = share / 8u / step * step;
        D.size = D.size < round ? round : D.size;
        D.size = D.size > most ? most : D.size;
    }
    D.n_items = n_items;
    D.n_chunks = n_items / D.size + (n_items % D.size != 0u ? 1u : 0u);
    D.per = (D.n_chunks + kXcds - 1u) / kXcds;
    D.apart = apart;
    return D;
}

// Chunks of XCD x's share.
__host__ __device__ inline uint32_t deal_share(const Deal &D, uint32_t x) {
    if (!D.apart) return (D.n_chunks + kXcds - 1u - x) / kXcds;
    const uint32_t lo = x * D.per, hi = lo + D.per;
    return (hi < D.n_chunks ? hi : D.n_chunks) - (lo < D.n_chunks ? lo : D.n_chunks);
}

// Items of chunk `at` of XCD x's share: the first, and in the upper half the
// end; 0 (an empty range) past the share's end.
__host__ __device__ inline unsigned long long deal_range(const Deal &D, uint32_t x, uint32_t at) {
    if (at >= deal_share(D, x)) return 0ull;
    const unsigned long long chunk = D.apart ? x * D.per + at : at * kXcds + x;
    const unsigned long long lo = chunk * D.size, hi = lo + D.size;
    return ((hi < D.n_items ? hi : D.n_items) << 32) | lo;
}

}  // namespace emt

#endif
