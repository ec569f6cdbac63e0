// How a work-group deals out its entries of the slow-tile list, on the CPU
// (test infrastructure: tests/test_host_deal.py compiles and runs it), with
// the function the trace kernel uses.  The work queue is dry, so a wave that
// gets no entry leaves for good; waves ask in any order.  Every entry has to be
// dealt exactly once, however uneven the sub-lists are.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "svo_internal.h"

int main(int argc, char** argv) {
    std::mt19937 g(argc > 1 ? (unsigned)std::atoi(argv[1]) : 1u);
    auto below = [&](uint32_t n) { return (uint32_t)(g() % n); };
    unsigned long dealt = 0, lists = 0, holes = 0;
    for (int it = 0; it < 4000; ++it) {
        const uint32_t wpb = 1 + below(16), blocks = 1 + below(it % 2 ? 40 : 512);
        uint32_t cnt[svo::kHotSub], longest = 0, want = 0;
        for (uint32_t& c : cnt) {
            const uint32_t kind = below(4);
            c = kind == 0 ? 0 : (kind == 1 ? below(8) : below(svo::kHotSubCap + 1));
            longest = std::max(longest, c);
            want += c;
        }
        const uint32_t n_deal = longest * svo::kHotSub;
        std::vector<uint8_t> seen(n_deal, 0);
        uint32_t got = 0;
        for (uint32_t b = 0; b < blocks; ++b) {
            uint32_t taken = 0;
            std::vector<uint32_t> waves(wpb);
            for (uint32_t w = 0; w < wpb; ++w) waves[w] = w;
            while (!waves.empty()) {
                const uint32_t at = below((uint32_t)waves.size());
                const uint32_t e = svo::hot_deal([&]() -> uint32_t { return taken++; }, wpb, blocks, b, n_deal, cnt);
                if (e == svo::kHotNone) {
                    waves.erase(waves.begin() + at);
                    continue;
                }
                if (e >= n_deal || e / svo::kHotSub >= cnt[e % svo::kHotSub] || seen[e]++) {
                    std::printf("entry %u dealt twice or past its sub-list\n", e);
                    return 1;
                }
                ++got;
            }
        }
        if (got != want) {
            std::printf("%u of %u entries dealt (%u work-groups of %u waves)\n", got, want, blocks, wpb);
            return 1;
        }
        dealt += got;
        holes += n_deal - want;
        ++lists;
    }
    std::printf("lists %lu dealt %lu holes %lu\n", lists, dealt, holes);
    return 0;
}
