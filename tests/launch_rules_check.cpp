// The rules that size a launch, on the host: prints "<rule> ok" or the first
// case that breaks the rule.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

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

// Every (head, slice) has one workgroup, and no XCD (32 CUs, a workgroup a CU;
// workgroups round-robin over 8) needs more rounds than dealing them out needs.
bool placement() {
    for (int H = 1; H <= 140; ++H)
        for (int per = 1; per <= 40; ++per) {
            const bool by_xcd = cap::heads_by_xcd(H, per);
            std::vector<int> seen((size_t)H * per), load(8);
            const unsigned grid = cap::head_slice_grid(H, per);
            for (unsigned b = 0; b < grid; ++b) {
                const cap::HeadSlice x = cap::head_slice(b, by_xcd, H, per);
                if (!x.on) continue;
                if (x.h < 0 || x.h >= H || x.slice < 0 || x.slice >= per) return std::printf("placement: %d x %d\n", H, per), false;
                ++seen[(size_t)x.h * per + x.slice];
                ++load[b % 8];
            }
            const int most = *std::max_element(load.begin(), load.end()), dealt = (H * per + 7) / 8;
            if (std::any_of(seen.begin(), seen.end(), [](int n) { return n != 1; }) || (most + 31) / 32 > (dealt + 31) / 32) {
                std::printf("placement: %d heads x %d slices: %d on one XCD\n", H, per, most);
                return false;
            }
        }
    return true;
}

}  // namespace

int main() {
    if (placement()) std::puts("placement ok");
    if (gather_shares()) std::puts("gather_shares ok");
    if (fp8_grid()) std::puts("fp8_grid ok");
    return 0;
}
