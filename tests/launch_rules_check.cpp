// The rules that size a launch, on the host: prints "<rule> ok" or the first
// case that breaks the rule.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
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
            if (per == 1 && grid != (unsigned)H) return std::printf("placement: %d workgroups for %d heads\n", grid, H), false;
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

cap::ScanParams call(int64_t T, int H, int dk, int dv, bool f32, bool states) {
    static float any;
    cap::ScanParams p{};
    p.T = T, p.H = H, p.dk = dk, p.dv = dv, p.in_f32 = f32, p.chunk_states = states ? &any : nullptr;
    return p;
}

// A call in segments: they cover the chunks, each has a chunk, the dk tokens of
// its hand-over where that lies in o, and the grid's arithmetic fits; with
// chunk states there are several.  Shapes whose pass was the faster one, by up
// to half, take the pass.
bool segments() {
    for (const int dk : {64, 128})
        for (int f32 = 0; f32 <= (dk == 64); ++f32)
            for (int states = 0; states < 2; ++states)
                for (int H = 1; H <= 300; H += H < 40 ? 1 : 13)
                    for (int dv = 16; dv <= 512; dv += 16)
                        for (const int64_t T : {0, 1, 65, 128, 511, 512, 1024, 1025, 1151, 1792, 2049, 3071, 4096, 6143, 8192, 16385, 1 << 20}) {
                            const cap::ScanParams p = call(T, H, dk, dv, f32, states);
                            if (!cap::linattn_in_segments(p)) continue;
                            const cap::SegPlan s = cap::linattn_seg_plan(p);
                            const int64_t n = (T + 63) / 64, last = (s.nseg - 1) * s.G * 64;
                            if (s.G < 1 || s.nseg < 1 || last >= T || s.nseg * s.G > 2 * n + s.G || (s.cols != 64 && s.cols != 128) ||
                                (s.cols == 128 && f32) || (states && s.nseg < 2) ||
                                (!states && s.nseg > 1 && (s.G * 64 < dk || T - last < dk))) {
                                std::printf("segments: %lld x %d x %d/%d\n", (long long)T, H, dk, dv);
                                return false;
                            }
                        }
    const int pass[][4] = {{2048, 48, 128, 80}, {2048, 18, 128, 208}, {4096, 25, 128, 144}, {4096, 40, 128, 96}, {4096, 14, 128, 144},
                           {8192, 21, 128, 176}, {16384, 24, 128, 144}, {16384, 18, 128, 176}, {1800, 32, 64, 64}, {4096, 40, 64, 80},
                           {8192, 32, 128, 128}, {2048, 64, 128, 128}, {981, 6, 128, 16}, {1129, 9, 128, 48}, {1366, 5, 128, 176}};
    for (const auto& c : pass)
        if (cap::linattn_in_segments(call(c[0], c[1], c[2], c[3], false, false))) {
            std::printf("segments: %d x %d x %d/%d is faster in one pass\n", c[0], c[1], c[2], c[3]);
            return false;
        }
    return true;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc == 7) {  // T H dk dv fp32 states: the plan of a linear-attention prefill
        const cap::ScanParams p = call(std::atoll(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]),
                                       std::atoi(argv[5]), std::atoi(argv[6]));
        const cap::SegPlan s = cap::linattn_seg_plan(p);
        if (cap::linattn_in_segments(p)) std::printf("%d %lld %lld\n", s.cols, (long long)s.nseg, (long long)s.G);
        else std::puts("one pass");
        return 0;
    }
    if (segments()) std::puts("segments ok");
    if (placement()) std::puts("placement ok");
    if (gather_shares()) std::puts("gather_shares ok");
    if (fp8_grid()) std::puts("fp8_grid ok");
    return 0;
}
