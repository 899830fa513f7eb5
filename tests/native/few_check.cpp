// Host-only check of the rule by which a call counts over binned cells or line
// grids (few_grains): equal views by their own seeds, mixed ones by the mean.
#include <cstdio>

#include "emt_dev.h"

using namespace emt;

static int failures = 0;

#define CHECK(cond)                                             \
    do {                                                        \
        if (!(cond)) {                                          \
            std::printf("FAIL line %d: %s\n", __LINE__, #cond); \
            ++failures;                                         \
        }                                                       \
    } while (0)

int main() {
    // grains, views with grains, seeds: the faster side where both were timed
    struct { unsigned long long n; uint32_t views; double seeds; bool cells; } timed[] = {
        {32 * 1800, 32, 32 * 123e3, true},   {32 * 1800, 32, 32 * 441e3, false},
        {75059, 1001, 4.65e6, true},         {335059, 1001, 23.0e6, true},
        {935059, 3001, 61.0e6, true},        {200059, 301, 16.6e6, true},
        {395059, 301, 35.9e6, true},         {1235059, 1001, 110.0e6, true},
        {215059, 101, 20.8e6, true},         {369999, 1001, 39.3e6, true},
        {86548, 65, 5.9e6, true},            {42430, 17, 3.94e6, true},
        {169999, 101, 37.6e6, false},        {89999, 21, 23.8e6, false},
        {47576, 11, 5.16e6, false},          {207781, 16, 26.4e6, false},
        {298298, 16, 52.2e6, false},         {27576, 1, 3.28e6, false},
        {320000, 64, 9.54e6, true},          {48000, 32, 9.28e6, false},
    };
    for (const auto &t : timed) CHECK(few_grains(t.n, t.views, -1, t.seeds / (double)t.n) == t.cells);
    // one large view among many small ones is no reason for grids of them all
    for (uint32_t small : {100u, 1000u, 30000u})
        CHECK(few_grains(35000 + 20ull * small, 1 + small, -1, 0.0) == (small >= 100));
    CHECK(!few_grains(35000, 1, -1, 0.0) && few_grains(8192, 1, -1, 0.0));
    CHECK(few_grains(900 * 48, 48, -1, 0.0) && !few_grains(3 * 27000, 3, -1, 0.0));
    CHECK(few_grains(0, 0, -1, 0.0) && few_grains(27000, 1, 999, 1e3) && !few_grains(27000, 1, 1000, 1e3));
    if (failures == 0) std::printf("few ok\n");
    return failures ? 1 : 0;
}
