// Work items shared out over the XCDs: every item is in one workgroup's share, and
// no workgroup has more than the items need: one while there is room for all, else
// the even share of its XCD.  Prints "ok" and returns 0.
#include <algorithm>
#include <cstdio>

#include "device.hpp"

using namespace qsv::dev;

int main() {
    for (uint64_t resident : {8, 256, 1024, 2048, 5})
        for (uint64_t items = 1; items <= 5000; items += items < 300 ? 1 : 37) {
            const unsigned grid = xcd_grid(items, resident), per = grid / kXcds;
            if (grid % kXcds || grid > std::max<uint64_t>(kXcds, resident)) {
                std::fprintf(stderr, "grid %u of %llu resident\n", grid, (unsigned long long)resident);
                return 1;
            }
            uint64_t seen = 0, longest = 0;
            for (unsigned w = 0; w < grid; ++w) {
                const uint64_t end = xcd_first(items, w % kXcds + 1);
                uint64_t mine = 0;
                for (uint64_t it = xcd_first(items, w % kXcds) + w / kXcds; it < end; it += per) ++mine;
                seen += mine;
                longest = std::max(longest, mine);
            }
            const uint64_t range = (items + kXcds - 1) / kXcds;
            if (seen != items || longest != (range + per - 1) / per ||
                (items + kXcds <= resident && longest != 1)) {
                std::fprintf(stderr, "%llu items, grid %u: %llu done, %llu in one workgroup\n",
                             (unsigned long long)items, grid, (unsigned long long)seen,
                             (unsigned long long)longest);
                return 1;
            }
        }
    std::printf("ok\n");
    return 0;
}
