// Every workgroup of the kernel that writes destinations in pairs gets a row and a pair of its own, and together they
// take every row of an item once for every pair.  The workgroups of an item taken by eighths have a tile each.
#include <cstdio>
#include <vector>

#include "../../paper_2511_06605_amd/csrc/dl_work.h"

int main()
{
    std::vector<uint32_t> sizes = {4089, 4095, 4096, 4097, 8191, 8192, 8193, 12288, 20000, 20001};
    for (uint32_t rows = 1; rows < 600; ++rows) sizes.push_back(rows);
    for (uint32_t rows : sizes)
        for (uint32_t pairs = 1; pairs <= 4; ++pairs) {
            std::vector<int> seen((size_t)rows * pairs, 0);
            std::vector<uint32_t> xcd(rows, ~0u);
            dl_fused_item item{};
            item.bytes = (uint64_t)rows << 10;
            item.k = 2 * pairs;
            const uint64_t blocks = dl_pair_blocks(item);
            if (blocks % 8) return 5;
            uint64_t idle = 0;
            for (uint32_t b = 0; b < blocks; ++b) {
                uint32_t row = ~0u, pair = ~0u;
                if (!dl_pair_locate(b, rows, pairs, &row, &pair)) {
                    ++idle;
                    continue;
                }
                if (row >= rows || pair >= pairs || seen[(size_t)pair * rows + row]++) {
                    std::printf("rows %u pairs %u block %u: row %u pair %u\n", rows, pairs, b, row, pair);
                    return 1;
                }
                // the workgroups of a row's pairs are dealt to the same one of eight XCDs
                if (xcd[row] == ~0u) xcd[row] = b % 8;
                if (xcd[row] != b % 8) {
                    std::printf("rows %u pairs %u row %u: XCDs %u and %u\n", rows, pairs, row, xcd[row], b % 8);
                    return 2;
                }
            }
            if (idle != blocks - (uint64_t)rows * pairs || idle > 7u * pairs) return 6;
            for (uint32_t b = (uint32_t)blocks; b < blocks + 10000; b += 9) {  // past the item
                uint32_t row, pair;
                if (dl_pair_locate(b, rows, pairs, &row, &pair)) return 7;
            }
        }
    for (uint32_t tiles = 1; tiles < 3000; ++tiles) {
        const uint32_t width = (uint32_t)dl_eighths_width(tiles);
        std::vector<int> seen(width, 0);
        if (width < tiles || width > tiles + 7) return 8;
        for (uint32_t b = 0; b < width; ++b) {
            const uint32_t t = dl_eighths_tile(b, width);
            if (t >= width || seen[t]++) return 9;
            if (t / (width / 8) != b % 8) return 10;  // an XCD's tiles lie together
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
