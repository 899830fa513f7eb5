// Host-only check of deal.h: whatever the number of items and the grid, the
// first chunks and those the counters hand out are every item once.
#include <cstdio>
#include <vector>

#include "deal.h"

using namespace emt;

static int failures = 0;

// Every workgroup's first range, then chunks from the counters, by the rule
// the kernel follows, workgroup by workgroup.
static void check(uint32_t n, uint32_t step, uint32_t waves, uint32_t grid, uint32_t most,
                  bool apart) {
    const Deal D = make_deal(n, step, waves, grid, most, apart);
    std::vector<uint8_t> taken(n, 0);
    unsigned long long total = 0;
    bool ok = D.size > 0;
    auto take = [&](unsigned long long r) {
        const uint32_t lo = (uint32_t)r, hi = (uint32_t)(r >> 32);
        for (uint32_t i = lo; i < hi && i < n; ++i) taken[i]++;
        ok = ok && lo < hi && hi <= n;
        total += hi - lo;
    };
    for (uint32_t b = 0; b < grid; ++b)
        if (const unsigned long long r = deal_range(D, b % kXcds, b / kXcds)) take(r);
    uint32_t counter[kXcds] = {};
    for (uint32_t b = 0; b < grid; ++b)
        for (uint32_t t = 0; t < kXcds; ++t) {
            const uint32_t x = (b + t) % kXcds;
            while (grid / kXcds + counter[x] < deal_share(D, x))
                if (const unsigned long long r = deal_range(D, x, grid / kXcds + counter[x]++))
                    take(r);
        }
    for (uint32_t i = 0; i < n; ++i) ok = ok && taken[i] == 1;
    if (!ok || total != n) {
        std::printf("FAIL n %u step %u grid %u apart %d: %llu items dealt\n", n, step, grid, apart,
                    total);
        ++failures;
    }
}

int main() {
    for (bool apart : {false, true})
        for (uint32_t grid : {8u, 512u, 1024u})
            for (uint32_t step : {16u, 17u, 64u})
                for (uint32_t n : {0u, 1u, 15u, 16u, 17u, 100u, 128u, 129u, 1000u, 2000u, 7168u,
                                   8192u, 8193u, 65535u, 100000u, 196607u, 196609u, 393215u,
                                   393217u, 1000003u, 5000011u})
                    check(n, step, 12, grid, 2048, apart);
    // the largest lists: shares add up to the chunks, and ranges stay 32-bit
    for (bool apart : {false, true})
        for (uint32_t n : {2147483647u, 4294967295u}) {
            const Deal D = make_deal(n, 64, 12, 512, 2048, apart);
            uint32_t chunks = 0;
            unsigned long long items = 0;
            for (uint32_t x = 0; x < kXcds; ++x) {
                chunks += deal_share(D, x);
                for (uint32_t at = 0; at < deal_share(D, x); ++at) {
                    const unsigned long long r = deal_range(D, x, at);
                    items += (r >> 32) - (uint32_t)r;
                }
            }
            if (chunks != D.n_chunks || items != n) {
                std::printf("FAIL n %u apart %d: %llu items\n", n, apart, items);
                ++failures;
            }
        }
    if (failures == 0) std::printf("deal ok\n");
    return failures ? 1 : 0;
}
