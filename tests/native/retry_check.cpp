// Host-only check of the capacity planner (capacity.h) where the members of all
// candidates are known although the candidates overflowed: whatever the first
// candidates held, the second attempt has room for all, and an eighth more.
#include <cstdio>

#include "capacity.h"

using namespace emt;

int main() {
    int failures = 0;
    for (uint32_t cand : {1025u, 5000u, 490471u, 2000000u})
        for (unsigned long long per : {4ull, 30ull, 60ull, 150ull}) {
            CapSizes c{1u << 20, 1024, 1u << 12};
            Ratios r{256.0, 8.0, 24.0};
            const Needs h{50000, per * cand, cand, true};
            if (h.members > kMemCapMax) continue;
            const bool ok = plan_retry(h, 16384, c, r) && fits(h, c);
            // no more than an eighth above what they need (or than the ratio
            // that the context starts with asks for)
            const double most = 1.126 * (per > 24 ? per : 24.0) * (cand + 1024.0) + 1024.0;
            // and the next such call starts with room for them, at no more a
            // candidate than these have (or the context starts with)
            const double each = per > 24 ? (double)per : 24.0, got = r.mem_per_cand;
            if (!ok || c.mem_cap > most || got > each || got * r.cand_per_grain * 16384 < h.members) {
                std::printf("FAIL %u candidates of %llu: members %u (at most %.0f), next %.1f each\n",
                            cand, per, c.mem_cap, most, got);
                ++failures;
            }
        }
    if (failures == 0) std::printf("retry ok\n");
    return failures ? 1 : 0;
}
