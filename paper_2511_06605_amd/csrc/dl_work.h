// Internal: the unit of device work and the geometry of cutting it into tiles.
// Shared by the host side (grid sizing) and the kernels (tile -> byte range) of
// the library, so both always agree.  Not part of the C boundary.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define DL_HD __host__ __device__ __forceinline__
#else
#define DL_HD inline
#endif

constexpr int DL_FAN = 8;  // destinations one work item can write from a single read

// A slot of device memory that the host fills through the BAR (short copy tables, masks): the payload, and in the
// last 8 bytes a stamp that is written after it.
constexpr uint32_t DL_PUSH_SLOT_BYTES = 64u << 10;
constexpr uint32_t DL_PUSH_PAYLOAD_BYTES = DL_PUSH_SLOT_BYTES - 8;

// What a kernel that reads a table written through the BAR needs besides the table: the stamp that the slot
// holds once the table is complete, how often to look for it, and where to report that it never came.
struct dl_pushed {
    uint64_t stamp;
    uint32_t tries;
    uint32_t pad;
    uint64_t *lost;  // host-coherent: the library's device error word
};

// Plain copy: one source, one destination.
struct dl_plain_item {
    const char *src;
    char *dst;
    uint64_t bytes;
};

// Swap (Sec. IV-C): the ranges [src, src + bytes) and [dst, dst + bytes), which
// do not overlap, exchange their contents.  Same layout and geometry as a plain
// copy; only what the device does with a tile differs.
struct dl_swap_item : dl_plain_item {};

// Fused broadcast copy: one source read once, k <= DL_FAN destinations.
struct dl_fused_item {
    const char *src;
    uint64_t bytes;
    uint32_t k;
    uint32_t pad;
    char *dst[DL_FAN];
};

// How an item is cut into tiles.  Tiles lie on a grid of DL_CUT bytes of the item's first destination: with
// shift = that address modulo DL_CUT, tile t of a tile size T (a multiple of DL_CUT) covers the item's bytes
// [t T - shift, (t + 1) T - shift), clipped to [0, bytes).  So every tile but an item's first begins on a
// DL_CUT boundary of the first destination, whatever the addresses are, and no two workgroups write into the
// same 128 bytes of it (partly written lines that two compute units share cost a third of the all-gather rate);
// the other destinations and the source may lie anywhere relative to that grid (16-byte accesses need no
// alignment on this hardware).
constexpr uint32_t DL_CUT = 128;

DL_HD uint32_t dl_item_shift(const dl_plain_item &it)
{
    return (uint32_t)((uint64_t)it.dst & (DL_CUT - 1u));
}

DL_HD uint32_t dl_item_shift(const dl_fused_item &it)
{
    return (uint32_t)((uint64_t)it.dst[0] & (DL_CUT - 1u));
}

// Number of tiles of an item (0 for an empty one).
template <class Item>
DL_HD uint64_t dl_item_tiles(const Item &it, uint32_t tile_bytes)
{
    if (it.bytes == 0) return 0;
    const uint64_t span = it.bytes + dl_item_shift(it);
    return span / tile_bytes + (span % tile_bytes ? 1u : 0u);
}

// Threads of a workgroup that moves plain copies, where the caller has not fixed them.  Beyond the launch-bound sizes
// a workgroup is one wavefront that moves one row, so consecutive rows of the address stream go to different XCDs.
// All-to-all between eight ranks with 512 KiB / 1 MiB / 4 MiB chunks, 256 threads against 64: 10.8 / 26.6 / 83.4 us
// against 10.6 / 24.0 / 79.7; at 256 KiB chunks (32 MiB moved) the larger workgroup is 1-3 % ahead when the buffers are in
// the caches and 8 % behind when they are not.  Not where the caller caps the number of workgroups (capped): there each
// makes many passes, and with a quarter of the wavefronts the 512 KiB / 2 MiB chunks took 51.9 / 250 us against 16.1 / 57.9
// (512 workgroups) and 16.1 / 78.4 against 8.8 / 36.2 (2048).
constexpr uint64_t DL_PLAIN_WAVE_MIN_BYTES = 48ull << 20;  // bytes moved (read + written)

DL_HD uint32_t dl_plain_threads(uint64_t moved, bool capped)
{
    return moved >= DL_PLAIN_WAVE_MIN_BYTES && !capped ? 64u : 256u;
}

// Workgroups of an item, a multiple of eight, and the tile of one of them where tiles next to each other share lines: the eight
// XCDs, to which workgroups are dealt in turn, take an eighth of the item each.
DL_HD uint64_t dl_eighths_width(uint64_t tiles) { return (tiles + 7u) & ~(uint64_t)7u; }
DL_HD uint32_t dl_eighths_tile(uint32_t wg, uint32_t width) { return (wg & 7u) * (width >> 3) + (wg >> 3); }

// Rows of 1 KiB that an item takes on that grid, and workgroups of the kernel that writes its destinations in pairs:
// as many for every pair, a multiple of eight (see dl_pair_locate).
DL_HD uint32_t dl_pair_rows(uint64_t bytes, uint32_t shift) { return (uint32_t)((bytes + shift + 1023u) >> 10); }
DL_HD uint64_t dl_pair_blocks(const dl_fused_item &it)
{
    return it.bytes ? (((uint64_t)dl_pair_rows(it.bytes, dl_item_shift(it)) + 7u) & ~(uint64_t)7u) * ((it.k + 1u) >> 1) : 0u;
}

// Row and pair of destinations of that kernel's workgroup `local` of an item of `rows` rows and `pairs` (1..4) pairs:
// the rows in chunks of DL_PAIR_ROWS, a chunk's rows for the first pair, then for the second, ...  A pair has a multiple
// of eight workgroups, also in an item's last chunk, so that a row's workgroups are dealt to the same one of eight XCDs
// and all but the first find it in that XCD's L2 (over eight ranks, 3 MiB + 1 KiB per rank: 35.0 us with the pairs
// 3073 workgroups apart, 30.3 with 3080).  False: one of the workgroups left over by that, or past the item.
// All-gather of 32 / 64 MiB per rank over eight ranks with chunks of 1024 rows 414 / 865 us, of 4096 370 / 747, of 8192
// 375 / 748, of 16 384 370 / 740, of 32 768 (as much source as the eight L2s hold) 419 / 842.
constexpr uint32_t DL_PAIR_ROWS = 4096;

DL_HD bool dl_pair_locate(uint32_t local, uint32_t rows, uint32_t pairs, uint32_t *row, uint32_t *pair)
{
    const uint32_t whole = local / DL_PAIR_ROWS;
    const uint32_t chunk = pairs == 3u ? whole / 3u : whole >> (pairs >> 1);  // (one, two or four pairs: a shift)
    const uint32_t row0 = chunk * DL_PAIR_ROWS;
    if (row0 >= rows) return false;
    const uint32_t left = (rows - row0 + 7u) & ~7u;
    const uint32_t n = left < DL_PAIR_ROWS ? left : DL_PAIR_ROWS;  // workgroups of a pair in this chunk
    const uint32_t in_chunk = local - row0 * pairs;
    *pair = (in_chunk >= n ? 1u : 0u) + (in_chunk >= 2u * n ? 1u : 0u) + (in_chunk >= 3u * n ? 1u : 0u);
    *row = row0 + (in_chunk - *pair * n);
    return *pair < pairs && *row < rows;
}

// Bytes [*lo, *hi) of an item that tile `tile` covers (*lo >= *hi: none).
DL_HD void dl_tile_range(uint32_t shift, uint64_t bytes, uint64_t tile, uint32_t tile_bytes, uint64_t *lo, uint64_t *hi)
{
    const uint64_t begin = tile * tile_bytes;  // on the grid; the item starts `shift` bytes into tile 0
    *lo = begin > shift ? begin - shift : 0;
    const uint64_t end = begin + tile_bytes - shift;
    *hi = end < bytes ? end : bytes;
}
