// Every workgroup of the kernel that writes destinations in pairs gets a row and a pair of its own, and together they
// take every row of an item once for every pair.
#include <cstdio>
#include <vector>

#include "../../paper_2511_06605_amd/csrc/dl_work.h"

int main()
{
    const uint32_t sizes[] = {1, 2, 4095, 4096, 4097, 8191, 8192, 8193, 12288, 20000};
    for (uint32_t rows : sizes)
        for (uint32_t pairs = 1; pairs <= 4; ++pairs) {
            std::vector<int> seen((size_t)rows * pairs, 0);
            for (uint32_t b = 0; b < rows * pairs; ++b) {
                uint32_t row = ~0u, pair = ~0u;
                if (!dl_pair_locate(b, rows, pairs, &row, &pair) || row >= rows || pair >= pairs || seen[(size_t)pair * rows + row]++) {
                    std::printf("rows %u pairs %u block %u: row %u pair %u\n", rows, pairs, b, row, pair);
                    return 1;
                }
            }
            // the workgroups of a row's pairs stay on one of eight XCDs where whole chunks allow it
            for (uint32_t b = 0; b + 4096 < rows * pairs && rows % 4096 == 0; ++b) {
                uint32_t r0, p0, r1, p1;
                dl_pair_locate(b, rows, pairs, &r0, &p0);
                dl_pair_locate(b + 4096, rows, pairs, &r1, &p1);
                if (p1 == p0 + 1 && r0 != r1) return 2;
            }
        }
    // shifts move an item over its grid: the number of rows is that of the bytes it touches
    for (uint64_t bytes = 1; bytes < 5000; ++bytes)
        for (uint32_t shift = 0; shift < DL_CUT; ++shift)
            if (dl_pair_rows(bytes, shift) != (shift + bytes - 1) / 1024 + 1) return 3;
    // a capped grid keeps its wavefronts, whatever the request moves
    for (uint64_t moved = 1; moved < 1ull << 40; moved *= 2)
        if (dl_plain_threads(moved, true) != 256u || dl_plain_threads(moved, false) != (moved < 48ull << 20 ? 256u : 64u)) return 4;
    std::puts("ok");
    return 0;
}
