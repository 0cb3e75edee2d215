// The rules that size a launch, on the host: prints "<rule> ok" or the first
// case that breaks the rule.
#include <cstdint>
#include <cstdio>

#include "internal.h"

namespace {

// Every block of a conversion has its place in the grid, whose threads along
// x stay below 2^32, and the blocks past the last are fewer than a row.
bool fp8_grid() {
    const uint64_t x0 = cap::kFp8GridX;
    for (const uint64_t base : {uint64_t(1), x0, 2 * x0, uint64_t(1) << 24, uint64_t(0x7fffffff)})
        for (int64_t d = -2; d <= 2; ++d) {
            const uint64_t blocks = base + (uint64_t)d;
            if (blocks == 0 || blocks > 0x7fffffff) continue;
            const uint64_t x = cap::fp8_grid_x((uint32_t)blocks), y = cap::fp8_grid_y((uint32_t)blocks);
            if (x * 256 > 0xffffffffu || y > 65535 || x * y < blocks || x * y - blocks >= x || (y > 1 && x != x0)) {
                std::printf("fp8_grid: %llu blocks: %llu x %llu\n", (unsigned long long)blocks, (unsigned long long)x,
                            (unsigned long long)y);
                return false;
            }
        }
    return true;
}

// Sharing sets in between the launches that it slowed down and those it helps
// (environments, bytes of a capsule).
bool gather_shares() {
    return !cap::gather_shares(16, 2363904) && !cap::gather_shares(40, 1184256) && !cap::gather_shares(31, 3543552) &&
           !cap::gather_shares(24, 4723200) && cap::gather_shares(31, 4723200) && cap::gather_shares(40, 3543552) &&
           cap::gather_shares(64, 2363904) && !cap::gather_shares(1, uint64_t(128) << 20);
}

}  // namespace

int main() {
    if (gather_shares()) std::puts("gather_shares ok");
    if (fp8_grid()) std::puts("fp8_grid ok");
    return 0;
}
