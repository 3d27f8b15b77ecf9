// Token dispatch placed on the device (Sec. IV-B: a token that goes to several experts is one source with several
// destinations).  Receive buffers are packed in token order, so where a token's row lands is a count: of the tokens
// before it that go to the same rank.  No copy list exists; every workgroup works out the places of its own tokens and
// copies their rows, in one launch:
//   - the mask on the host: the host packs it to a byte per token and counts the rows taken before every group of 64
//     tokens (control work, Sec. III-B2, done where the mask is); both travel in the kernel arguments (up to 2048
//     tokens), or through the BAR, or, where that way is not open, in the arguments of several launches.  (Fewer than 256
//     tokens off the grid are lowered to a list on the host after all, see OFF_GRID_MIN_TOKENS);
//   - the mask in device memory: every workgroup counts the tokens in front of its own group itself (at most 80 KiB
//     of mask, which the L2 holds); or, for a large request, a first kernel packs the groups (see PACK_FIRST_BYTES).
// Inside a group of 64 the places come from one ballot per rank.
//
// Before, a kernel built a table of 88-byte items from the mask (and another counted for it) and the row kernel for
// long lists read the table back, one workgroup of two wavefronts per 1 KiB row.  Rows of 14 336 bytes, call to call:
// 128 tokens per rank (93 MB moved) with the mask on the host 25.1 us in two launches, now 13.8 in one, with the mask
// on the device 28.4 (three launches) and 14.3; 512 per rank (370 MB) 72.6 : 55.4 and 75.7 : 57.0 (6.5 TB/s).
#include "dl_device.h"
#include "dl_internal.h"

#include <string.h>

namespace {

constexpr int DISPATCH_W = 8;              // ranks this path handles: exactly 8 (one 64-bit mask word per token)
constexpr uint32_t GROUP = 64;             // tokens whose places one wavefront's ballots tell apart
constexpr uint32_t DISPATCH_GROUPS = 32;   // groups per launch with the mask in the kernel arguments (3.2 KiB of the 4 KiB they may take)
constexpr uint32_t MAX_WAVES = 8;          // wavefronts of a workgroup
constexpr uint64_t ALONE_MAX_TOKENS = 512;     // tokens up to which a workgroup is one wavefront (see dispatch_setup),
constexpr uint64_t ALONE_LIST_MAX_ROWS = 3400; // ... and 1 KiB rows, with the mask on the host
constexpr uint64_t ALONE_MASK_MAX_ROWS = 8192; // ... and in device memory

struct dispatch_args {
    const char *in[DISPATCH_W];
    char *out[DISPATCH_W];
    uint32_t first_token[DISPATCH_W];  // tokens before rank i
    uint32_t tokens;                   // over all ranks
    uint32_t token0;                   // of them, where this launch begins (a multiple of GROUP)
    uint64_t row_bytes;
    uint32_t token_waves;              // wavefronts that share a token's rows
    uint32_t wg_tokens;                // tokens of a workgroup (a power of two, at most GROUP)
};

struct dispatch_group {
    uint32_t taken[DISPATCH_W];  // rows that earlier groups' tokens take in each receive buffer
    uint8_t ranks[GROUP];        // bit j: the token goes to rank j
};

struct dispatch_list {
    dispatch_args a;
    dispatch_group group[DISPATCH_GROUPS];
};
static_assert(sizeof(dispatch_list) <= 4096, "kernel arguments");
static_assert(sizeof(dispatch_group) % 16 == 0, "whole words");

// Where the row of token `token` (< a.tokens) begins: its rank is the last one that starts at or before it.
__device__ __forceinline__ const char *dl_dispatch_source(const dispatch_args &a, uint32_t token)
{
    const char *src = a.in[0];
    uint32_t first = 0;
#pragma unroll
    for (int r = 1; r < DISPATCH_W; ++r)
        if (a.first_token[r] <= token) {
            src = a.in[r];
            first = a.first_token[r];
        }
    return src + (uint64_t)(token - first) * a.row_bytes;
}

// On the grid (see dl_rows_body): what one wavefront copies of a token's row, 1 KiB rows `row0`, row0 + stride, ...,
// ROWS of them.  Every row is loaded once, into registers, as soon as the token is known; the loads are in
// flight while the wavefront finds out where the row goes (128 tokens per rank, mask on the device: 18.1 -> 16.4 us).
// AHEAD: what decides where the row goes comes from memory too, and is worked on before the row is waited for.  Then every
// lane loads, past the row's end its first 16 bytes: with loads that some path leaves out the compiler cannot tell how many
// are outstanding, and waits for the row together with whatever was asked for in front of it.
template <int POL, int ROWS, bool AHEAD = false>
struct dispatch_row {
    const char *src;
    uint64_t bytes;
    uint32_t row0, stride;
    dl_u32x4 v[ROWS];

    __device__ __forceinline__ uint64_t byte(int i) const
    {
        return ((uint64_t)(row0 + (uint32_t)i * stride) << 10) + ((threadIdx.x & 63u) << 4);
    }
    __device__ __forceinline__ void load(const dispatch_args &a, uint32_t token, uint32_t first_row)
    {
        src = dl_dispatch_source(a, token);
        bytes = a.row_bytes;
        row0 = first_row;
        stride = a.token_waves;
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
            if (AHEAD || byte(i) < bytes) v[i] = dl_ld16<POL>(src + (byte(i) < bytes ? byte(i) : 0));
    }
    // The token is number `in_group` of the 64 whose ranks the lanes hold in `mine`; `taken(j)` rows were placed in
    // receive buffer j before the group.
    template <class Taken>
    __device__ __forceinline__ void store(const dispatch_args &a, uint32_t in_group, uint32_t mine, Taken taken) const
    {
        const uint64_t before = (1ull << in_group) - 1ull;
        char *d[DISPATCH_W];
        if constexpr (AHEAD) {
#pragma unroll
            for (int j = 0; j < DISPATCH_W; ++j) {
                const uint64_t votes = __ballot((mine >> j) & 1u);
                d[j] = (votes >> in_group) & 1u ? a.out[j] + (uint64_t)(taken(j) + (uint32_t)__popcll(votes & before)) * bytes : nullptr;
            }
            arrived();
        }
#pragma unroll
        for (int j = 0; j < DISPATCH_W; ++j) {
            if constexpr (AHEAD) {
                if (!d[j]) continue;
            } else {
                const uint64_t votes = __ballot((mine >> j) & 1u);
                if (!((votes >> in_group) & 1u)) continue;
                d[j] = a.out[j] + (uint64_t)(taken(j) + (uint32_t)__popcll(votes & before)) * bytes;
            }
#pragma unroll
            for (int i = 0; i < ROWS; ++i)
                if (byte(i) < bytes) dl_st16<POL>(d[j] + byte(i), v[i]);
        }
    }
    // One wait for the whole row: at each use it would be waited for together with the stores in between.
    __device__ __forceinline__ void arrived() const
    {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) asm volatile("" ::"v"(v[i]));
    }
};

// Off the grid the destinations of a row lie differently against each other, and stores across 16-byte boundaries go to
// memory in pieces (rows of 14 338 bytes, 512 tokens per rank: 103 us with one load and unaligned stores), so every 1 KiB
// row is one plain copy per destination, each cut on its own grid; its loads after the first one hit the caches.
// What a small request takes here is instructions: a row and a destination are about a hundred of them, of one wavefront
// and fetched anew by every kernel.  So the destinations are a loop that is not unrolled, over those that the token goes
// to (mask on the host, 8 tokens per rank, rows of 14 338 / 16 400 bytes: 10.0 / 7.5 us unrolled eightfold, 7.2 / 5.5 as
// a loop; four or eight destinations' loads in flight together: 9.6 / 7.3, and 102 instead of 79 us at 512 per rank).
// Called by a wavefront for rows row0, row0 + a.token_waves, ..., ROWS of them, of token `token`, number `in_group` of
// the 64 whose ranks the lanes hold in `mine`; `taken(j)` rows were placed in receive buffer j before the group.
template <int POL, int ROWS, class Taken>
__device__ __forceinline__ void dl_dispatch_off_grid(const dispatch_args &a, uint32_t token, uint32_t in_group, uint32_t row0, uint32_t mine,
                                                     Taken taken)
{
    const char *const src = dl_dispatch_source(a, token);
    const uint64_t before = (1ull << in_group) - 1ull, bytes = a.row_bytes;
    const uint32_t ranks = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)in_group);
#pragma unroll 1
    for (uint32_t left = ranks; left; left &= left - 1u) {
        const uint32_t j = (uint32_t)__builtin_ctz(left);
        const uint64_t votes = __ballot((mine >> j) & 1u);
        const dl_plain_item it{src, a.out[j] + (uint64_t)(taken(j) + (uint32_t)__popcll(votes & before)) * bytes, bytes};
#pragma unroll 1
        for (int i = 0; i < ROWS; ++i) {
            const uint64_t row = row0 + (uint32_t)i * a.token_waves;
            if ((row << 10) >= bytes + DL_CUT) break;  // past the end wherever on its grid the copy begins
            dl_plain_row<POL, false>(it, row);
        }
    }
}

// Wavefront -> its token of the workgroup, and its first row.
template <int ROWS>
__device__ __forceinline__ void dl_dispatch_place(const dispatch_args &a, uint32_t *token_in_wg, uint32_t *row0)
{
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t t = 0, w = wave;
    while (w >= a.token_waves) {  // (at most MAX_WAVES rounds)
        w -= a.token_waves;
        ++t;
    }
    *token_in_wg = t;
    *row0 = blockIdx.x * a.token_waves * ROWS + w;
}

// A wavefront's rows of token `token`, whose group's record is g.
template <int POL, bool ON_GRID, int ROWS>
__device__ __forceinline__ void dl_dispatch_group_rows(const dispatch_args &a, const dispatch_group &g, uint32_t token, uint32_t row0)
{
    const uint32_t mine = g.ranks[threadIdx.x & 63u];
    const auto taken = [&](uint32_t j) { return g.taken[j]; };
    if constexpr (ON_GRID) {
        dispatch_row<POL, ROWS> row;
        row.load(a, token, row0);
        row.store(a, token % GROUP, mine, taken);
    } else {
        dl_dispatch_off_grid<POL, ROWS>(a, token, token % GROUP, row0, mine, taken);
    }
}

template <int POL, bool ON_GRID, int ROWS>
__global__ void __launch_bounds__(64 * MAX_WAVES) dl_dispatch_list_kernel(const dispatch_list p)
{
    uint32_t t, row0;
    dl_dispatch_place<ROWS>(p.a, &t, &row0);
    const uint32_t first = blockIdx.y * p.a.wg_tokens;  // within this launch
    const uint32_t token = p.a.token0 + first + t;
    if (token < p.a.tokens) dl_dispatch_group_rows<POL, ON_GRID, ROWS>(p.a, p.group[first / GROUP], token, row0);
}

// The groups in device memory, written there by the kernel in front (dl_dispatch_pack_kernel).
template <int POL, bool ON_GRID, int ROWS>
__global__ void __launch_bounds__(64 * MAX_WAVES) dl_dispatch_packed_kernel(const dispatch_args a, const dispatch_group *__restrict__ groups)
{
    uint32_t t, row0;
    dl_dispatch_place<ROWS>(a, &t, &row0);
    const uint32_t token = blockIdx.y * a.wg_tokens + t;
    if (token < a.tokens) dl_dispatch_group_rows<POL, ON_GRID, ROWS>(a, groups[token / GROUP], token, row0);
}

// The groups in device memory, written there by the host through the BAR just before the launch: read past the caches,
// once the slot's stamp has been seen (see dl_pushed_entry in the row kernels), and handed on through LDS.
template <int POL, bool ON_GRID, int ROWS>
__global__ void __launch_bounds__(64 * MAX_WAVES) dl_dispatch_pushed_kernel(const dispatch_args a, const dispatch_group *groups,
                                                                            const dl_pushed ps)
{
    constexpr uint32_t WORDS = sizeof(dispatch_group) / 8;
    __shared__ uint64_t raw[WORDS];
    __shared__ uint32_t sealed;
    uint32_t t, row0;
    dl_dispatch_place<ROWS>(a, &t, &row0);
    const uint32_t first = blockIdx.y * a.wg_tokens;
    const bool valid = first + t < a.tokens;  // uniform over the wavefront
    if (threadIdx.x == 0) sealed = dl_pushed_sealed(groups, ps) ? 1u : 0u;
    __syncthreads();
    if (!sealed) {
        if (threadIdx.x == 0) dl_pushed_report_lost(ps);  // nothing copied by this workgroup; the host hears of it
        return;
    }
    if (threadIdx.x < WORDS) raw[threadIdx.x] = dl_ld<DL_POL_COHERENT>(dl_global<uint64_t>(groups + first / GROUP) + threadIdx.x);
    dispatch_row<POL, ROWS> row;
    if constexpr (ON_GRID)
        if (valid) row.load(a, first + t, row0);
    __syncthreads();
    if (!valid) return;
    const dispatch_group &g = *reinterpret_cast<const dispatch_group *>(raw);
    const uint32_t mine = g.ranks[threadIdx.x & 63u];
    const auto taken = [&](uint32_t j) { return (uint32_t)__builtin_amdgcn_readfirstlane(g.taken[j]); };
    if constexpr (ON_GRID)
        row.store(a, (first + t) % GROUP, mine, taken);
    else
        dl_dispatch_off_grid<POL, ROWS>(a, first + t, (first + t) % GROUP, row0, mine, taken);
}

// Every byte of half a mask word to 0 or 1: adding 0x7f to its low seven bits carries into the eighth unless they are 0.
// keep: what of the result counts.
__device__ __forceinline__ uint32_t dl_mask_fold(uint32_t w, uint32_t keep = 0x01010101u)
{
    return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) >> 7 & keep;
}

// Sum over the wavefront, which lane 63 has: within rows of 16 lanes by shifts, then from row to row, all in the vector ALU
// (shuffles go through the LDS, whose pipe the wavefronts of a compute unit share).
__device__ __forceinline__ uint32_t dl_wave_sum63(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return x;
}

// The mask in device memory: how many rows the tokens in front of a group take in each receive buffer, and the ranks of
// the group's own token `lane` (0 past the last one).  Counted by the whole workgroup; `rows` runs behind the first
// loads, which are in flight meanwhile, or (ROWS_FIRST) in front of them.
struct dispatch_counts {
    uint32_t c[4];  // 16 bits a rank: ranks 0|2, 1|3, 4|6, 5|7
    uint32_t mine;

    // For a j that is known when the code is compiled.
    __device__ __forceinline__ uint32_t taken(uint32_t j) const
    {
        const uint32_t both = c[(j >> 2) * 2u + (j & 1u)];
        return (j & 2u) ? both >> 16 : both & 0xFFFFu;
    }
    // For any other: four ranks a word, in their order, and a shift.  (An array that j indexes would be kept in memory, and
    // all that depends on it counted as different for every lane.)
    struct packed {
        uint64_t ranks0, ranks4;
        __device__ __forceinline__ uint32_t taken(uint32_t j) const { return (uint32_t)((j < 4u ? ranks0 : ranks4) >> (16u * (j & 3u))) & 0xFFFFu; }
    };
    __device__ __forceinline__ packed pack() const
    {
        const auto four = [](uint32_t even, uint32_t odd) {
            return (uint64_t)((even & 0xFFFFu) | (odd << 16)) | (uint64_t)((even >> 16) | (odd & 0xFFFF0000u)) << 32;
        };
        return packed{four(c[0], c[1]), four(c[2], c[3])};
    }
    template <bool ROWS_FIRST, class Rows>
    __device__ __forceinline__ void count(const uint8_t *mask, uint32_t tokens, uint32_t group0, Rows rows)
    {
        __shared__ uint32_t part[MAX_WAVES][4];
        const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t waves = blockDim.x >> 6;
        // (the last group's lanes past the last token read that one's word)
        uint64_t own = dl_global<uint64_t>(mask)[group0 + lane < tokens ? group0 + lane : tokens - 1u];
        // two tokens per 16-byte load, up to BATCH loads in flight; a thread sums at most DL_DISPATCH_DEVICE_MAX_TOKENS / 64
        // words, so a byte of the sum does not overflow
        static_assert(DL_DISPATCH_DEVICE_MAX_TOKENS / 64 <= 255, "bytewise sums");
        constexpr uint32_t BATCH = 6;
        const uint32_t step = 2u * blockDim.x, i0 = 2u * threadIdx.x;
        dl_u32x4 w[BATCH];
        // Lanes past the group's beginning load the mask's first words (group0 is a multiple of GROUP: there are any) and count none
        // of them, loads that no lane needs are left out for all: whether a load is outstanding then depends on no lane.
        const auto fetch = [&](uint32_t base) {
#pragma unroll
            for (uint32_t u = 0; u < BATCH; ++u) {
                const uint32_t i = base + i0 + u * step;
                if (base + u * step < group0) w[u] = dl_ld16<DL_POL_WT>((const char *)mask + 8ull * (i < group0 ? i : 0u));
            }
        };
        uint32_t lo = 0, hi = 0;
        const auto add = [&](uint32_t base) {
#pragma unroll
            for (uint32_t u = 0; u < BATCH; ++u) {
                if (base + u * step >= group0) break;
                const uint32_t keep = base + i0 + u * step < group0 ? 0x01010101u : 0u;
                lo += dl_mask_fold(w[u].x, keep) + dl_mask_fold(w[u].z, keep);
                hi += dl_mask_fold(w[u].y, keep) + dl_mask_fold(w[u].w, keep);
            }
        };
        if constexpr (ROWS_FIRST) rows();
        fetch(0);
        if constexpr (!ROWS_FIRST) rows();
        add(0);
        for (uint32_t base = BATCH * step; base < group0; base += BATCH * step) {
            fetch(base);
            add(base);
        }
        // to 16 bits a rank, two ranks a word
        c[0] = lo & 0x00FF00FFu;
        c[1] = (lo >> 8) & 0x00FF00FFu;
        c[2] = hi & 0x00FF00FFu;
        c[3] = (hi >> 8) & 0x00FF00FFu;
        static_assert(DL_DISPATCH_DEVICE_MAX_TOKENS < 65536, "16-bit counts");
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] = dl_wave_sum63(c[q]);
        if (waves == 1u) {
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = (uint32_t)__builtin_amdgcn_readlane((int)c[q], 63);
        } else {
            if (lane == 63u) {
#pragma unroll
                for (int q = 0; q < 4; ++q) part[wave][q] = c[q];
            }
            __syncthreads();
            // a lane per word, rows of four wavefronts summed by shifts
            static_assert(MAX_WAVES * 4 <= 32, "two rows of lanes");
            uint32_t x = lane < 4u * waves ? part[lane >> 2][lane & 3u] : 0u;
            x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
            x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
#pragma unroll
            for (int q = 0; q < 4; ++q)
                c[q] = (uint32_t)__builtin_amdgcn_readlane((int)x, 12 + q) + (uint32_t)__builtin_amdgcn_readlane((int)x, 28 + q);
        }
        asm volatile("" : "+v"(own));  // not looked at (and so waited for) earlier
        const uint32_t low = dl_mask_fold((uint32_t)own), high = dl_mask_fold((uint32_t)(own >> 32));
        // four low bits into the top four: the multiplication moves bit 8 j to bit 24 + j
        mine = group0 + lane < tokens ? ((low * 0x01020408u) >> 24 & 0xFu) | ((high * 0x01020408u) >> 20 & 0xF0u) : 0u;
    }
};

// What bounds it beyond its bytes: the counting, by every workgroup, in front of the first store.  It runs while the row is on
// its way, in the vector ALU alone (shuffles of a whole compute unit's wavefronts kept the LDS busy for 1 us a pass).  Row
// waited for first and sums by shuffles : this, one mask and set of buffers after the other in a graph, 2 / 16 / 64 tokens per
// rank of 4 KiB 4.2 / 4.3 / 5.2 : 2.9 / 3.2 / 4.1 us, of 14 KiB 4.2 / 5.1 / 9.2 : 2.9 / 3.9 / 8.3; in a stream of launches 128 /
// 253 per rank of 4 KiB 7.3 / 9.9 : 6.9 / 8.7, 192 / 253 / 512 of 14 KiB 25.6 / 32.1 / 59.3 : 23.0 / 29.2 / 57.1 (6.4 TB/s).
template <int POL, bool ON_GRID, int ROWS>
__global__ void __launch_bounds__(64 * MAX_WAVES) dl_dispatch_mask_kernel(const dispatch_args a, const uint8_t *__restrict__ mask)
{
    uint32_t t, row0;
    dl_dispatch_place<ROWS>(a, &t, &row0);
    const uint32_t first = blockIdx.y * a.wg_tokens;
    const uint32_t group0 = first & ~(GROUP - 1u);  // the same for the whole workgroup: wg_tokens divides GROUP
    const bool valid = first + t < a.tokens;  // uniform over the wavefront
    // all arguments in one go, in front of everything (left to itself the compiler asks for each where it is used, a
    // scalar round trip every time: 1 / 128 / 512 tokens per rank 6.1 / 14.3 / 58.7 us against 5.8 / 14.0 / 58.3)
    if constexpr (ON_GRID)
        asm volatile("" ::"s"(a.in[0]), "s"(a.in[1]), "s"(a.in[2]), "s"(a.in[3]), "s"(a.in[4]), "s"(a.in[5]), "s"(a.in[6]),
                     "s"(a.in[7]), "s"(a.out[0]), "s"(a.out[1]), "s"(a.out[2]), "s"(a.out[3]), "s"(a.out[4]), "s"(a.out[5]),
                     "s"(a.out[6]), "s"(a.out[7]), "s"(a.row_bytes), "s"(a.first_token[1]), "s"(a.first_token[2]),
                     "s"(a.first_token[3]), "s"(a.first_token[4]), "s"(a.first_token[5]), "s"(a.first_token[6]),
                     "s"(a.first_token[7]));
    dispatch_row<POL, ROWS, true> row;
    dispatch_counts c;
    // The rows are loaded behind the mask's first loads: those come back first, and are counted meanwhile.  But where the loads
    // stream, all rows of a workgroup are waited for there: loads in one burst and stores in the next are then the faster order
    // (see dispatch_setup).  With eight wavefronts of two rows, rows of up to 2 KiB and of more than 16, the burst lies in front
    // of the mask's loads, which held some rows up until others were being stored.  Behind : in front, one buffer set / three / sets
    // that fit no cache, 650 per rank of 2 KiB 11.1 / 12.8 / 15.6 : 11.2 / 11.5 / 14.2 us, 900 14.3 / 18.9 / 22.6 : 14.5 / 16.7 / 19.7; 75 of
    // 18 KiB 11.4 / 12.5 / 14.2 : 11.5 / 11.8 / 14.2, 85 12.2 / 14.5 / 16.9 : 12.5 / 14.6 / 17.2, 56 of 32 KiB 13.3 / 15.9 / 19.0 : 13.3 / 14.6 /
    // 18.2 (without a burst 650 of 2 KiB 10.9 / 13.6 / 15.8, 85 of 18 KiB 12.5 / 15.2 / 18.1, 56 of 32 KiB 13.4 / 17.1 / 20.9).
    constexpr bool BURST = POL == DL_POL_STREAM_IN;
    c.count<BURST && ROWS == 2>(mask, a.tokens, group0, [&] {
        if constexpr (ON_GRID) {
            row.load(a, valid ? first + t : a.tokens - 1u, row0);
            if constexpr (BURST) row.arrived();
        }
    });
    if (!valid) return;
    if constexpr (ON_GRID) {
        row.store(a, first + t - group0, c.mine, [&](uint32_t j) { return c.taken(j); });
    } else {
        const auto before = c.pack();
        dl_dispatch_off_grid<POL, ROWS>(a, first + t, first + t - group0, row0, c.mine, [&](uint32_t j) { return before.taken(j); });
    }
}

// One workgroup per group: its record, for dl_dispatch_packed_kernel.
__global__ void __launch_bounds__(64 * MAX_WAVES) dl_dispatch_pack_kernel(const uint8_t *__restrict__ mask, uint32_t tokens, dispatch_group *groups)
{
    dispatch_counts c;
    c.count<false>(mask, tokens, blockIdx.x * GROUP, [] {});
    dispatch_group &g = groups[blockIdx.x];
    if (threadIdx.x < GROUP) g.ranks[threadIdx.x] = (uint8_t)c.mine;
    if (threadIdx.x < (uint32_t)DISPATCH_W) g.taken[threadIdx.x] = c.pack().taken(threadIdx.x);
}

// How far behind a DL_CUT boundary the first destination of a row can lie: rows stand whole multiples of
// row_bytes into the receive buffers, so every such address is a multiple of the largest power of two that
// divides row_bytes and all of the buffers' addresses.
uint32_t worst_shift(void *const *out, int W, size_t row_bytes)
{
    uint64_t m = row_bytes;
    for (int i = 0; i < W; ++i) m |= (uint64_t)out[i];
    m &= DL_CUT - 1u;
    return m ? DL_CUT - (uint32_t)(m & (0 - m)) : 0u;
}

// Every row lies as the on-grid instance of the row kernel wants it (see dl_rows_body).
bool rows_on_grid(const void *const *in, void *const *out, int W, size_t row_bytes)
{
    uint64_t m = row_bytes & 3u;
    for (int i = 0; i < W; ++i) m |= (uint64_t)in[i] & 3u;
    return m == 0 && (row_bytes & 15u) == 0 && worst_shift(out, W, row_bytes) == 0;
}

// What the kernels are told, and their grid: a token's rows are shared out over up to MAX_WAVES wavefronts (a longer
// row takes several workgroups, blockIdx.x); short rows put several tokens into a workgroup.
struct dispatch_shape {
    uint32_t grid_x;
    uint32_t threads;
    int policy;
    bool on_grid;
    bool long_rows;  // longer than a workgroup holds
    int rows;        // of a wavefront, in flight together
};

// Calls f with the cache policy, whether all lies on the grid, and the rows of a wavefront as compile-time constants.
template <class F>
void with_instance(const dispatch_shape &sh, F f)
{
    dl_with_policy_and_grid(sh.policy, sh.on_grid, [&](auto pol, auto og) {
        if constexpr (decltype(og)::value) {  // off the grid a wavefront's rows are a loop, and two of them enough
            if (sh.rows == 3) return f(pol, og, std::integral_constant<int, 3>{});
            if (sh.rows == 4) return f(pol, og, std::integral_constant<int, 4>{});
        }
        if (sh.rows == 1)
            f(pol, og, std::integral_constant<int, 1>{});
        else
            f(pol, og, std::integral_constant<int, 2>{});
    });
}

int dispatch_setup(const void *const *in, void *const *out, const uint32_t *tokens, uint64_t total, size_t row_bytes,
                   bool mask_on_device, dispatch_args *a, dispatch_shape *sh)
{
    uint32_t first = 0;
    for (int i = 0; i < DISPATCH_W; ++i) {
        a->in[i] = (const char *)in[i];
        a->out[i] = (char *)out[i];
        a->first_token[i] = first;
        first += tokens[i];
    }
    a->tokens = (uint32_t)total;
    a->token0 = 0;
    a->row_bytes = row_bytes;
    const uint64_t rows = (row_bytes + worst_shift(out, DISPATCH_W, row_bytes) + 1023u) >> 10;
    if (rows * total >= (1ull << 30)) return DL_ERR_INVALID;  // beyond a grid
    sh->on_grid = rows_on_grid(in, out, DISPATCH_W, row_bytes);
    // Cache policy by an upper bound of what is moved (every token to every rank; top-8 of 256 experts: two thirds of
    // that), at the lines of the fan-outs of a list: write-through stores, with streaming loads, streamed output.
    // 128 tokens of 14 336 bytes per rank (126 MiB by this measure) 15.8 / 15.3 / 17.1 us, 512 (504 MiB) 70.6 / 71.8 / 58.6.
    const uint64_t bound = total * row_bytes * (1u + DISPATCH_W);
    const dl_config &c = g_dl.cfg;
    sh->policy = bound >= c.nontemporal_min_bytes ? DL_POL_STREAM
                 : bound > c.write_through_max_bytes ? DL_POL_STREAM_OUT : bound >= DL_FAN_STREAM_IN_MIN_BYTES ? DL_POL_STREAM_IN : DL_POL_WT;
    // Rows of a wavefront, (at most) wavefronts of a workgroup.  Off the grid, rows that one workgroup can hold: a row per wavefront
    // while the chip has room for all of them (8 tokens of 14 338 bytes per rank 7.2 us against 10.5 with two), else two
    // (1024 per rank, sources not in the caches: 184 us against 202).  Longer rows: four wavefronts of a row each
    // (16 400 bytes, 1024 per rank, likewise 189 us against 228 with eight of two; 300 000 bytes, 32 per rank 65 against 75).
    const uint64_t in_one = 2u * MAX_WAVES;
    uint32_t waves = MAX_WAVES;
    sh->rows = 2;
    sh->long_rows = rows > in_one;
    if (!sh->on_grid && sh->long_rows) {
        waves = 4;
        sh->rows = 1;
    } else if (!sh->on_grid) {
        if (rows == 1 || rows * total <= 8192u) sh->rows = 1;
    } else if (sh->policy == DL_POL_STREAM_OUT && !mask_on_device) {
        // Large requests on the grid: two wavefronts of a row each.  Consecutive rows then go to different XCDs, and fewer
        // destinations are written at once by each.  Rows of 14 336 bytes, 512 / 1024 per rank 58.5 / 140 us with eight
        // wavefronts of two rows, 54.6 / 125 this way; of 64 KiB, sources not in the caches, 256 / 512 / 1024 per rank
        // 163 / 320 / 638 and 141 / 278 / 564.  Smaller requests stay: 128 per rank of 14 336 bytes 13.0 and 17.9.
        // (Not where every workgroup counts the mask: four times as many workgroups, 512 per rank of 64 KiB 378 us.)
        waves = 2;
        sh->rows = 1;
    } else if (sh->policy == DL_POL_WT && total <= ALONE_MAX_TOKENS &&
               rows * total <= (mask_on_device ? ALONE_MASK_MAX_ROWS : ALONE_LIST_MAX_ROWS)) {
        // Small: a wavefront by itself, so that nothing waits for a neighbour and a wavefront has the fewest instructions
        // to fetch.  Eight wavefronts of two rows : this, mask on the host, in a graph: up to a row for each of the chip's 1024 SIMDs
        // always (64 tokens per rank of 2 KiB 2.87 : 2.52 us, 32 of 4 KiB 2.90 : 2.52, 16 of 8 KiB 2.94 : 2.53), up to two with sets that
        // fit no cache (48 of 3 KiB 3.95 : 3.69, 40 and 64 of 4 KiB 4.32 : 3.78 and 4.65 : 4.42, 40 of 5 KiB 4.21 : 4.06) and rows of 8 KiB and more
        // (24 of 8 KiB 3.07 : 2.98, 20 of 12 KiB 3.20 : 3.08), while shorter rows in the caches, which then go two by two in one
        // round, lose (48 of 3 KiB 2.67 : 2.89, 64 of 4 KiB 3.22 : 3.30, 40 of 5 KiB 2.88 : 3.10); beyond that mostly again (64 of 6 KiB
        // 3.93 : 3.85 and 5.52 : 5.30, 40 of 8 KiB 3.63 : 3.57 and 5.15 : 4.85, 40 of 10 KiB 4.44 : 3.94 and 6.02 : 5.48), to 3400 rows
        // (56 of 8 KiB 4.32 : 4.32, 44 of 10 KiB 4.55 : 4.55; 57 of 10 KiB, three sets in turn, 6.5 : 7.5); 128 of 4 KiB 4.94 : 5.03.
        // Mask on the device, 16 / 64 per rank of 4 KiB 4.96 : 4.01 and 5.41 : 4.96, of 8 KiB 5.12 : 4.23 and 6.90 : 6.34, of
        // 14 KiB 6.19 : 4.71 and 10.3 : 9.2 (with two rows; 9.7 with one); there every wavefront counts the mask for itself
        // (128 of 4 KiB 6.8 : 7.3), and 512 tokens of 20 rows take 12.5 : 13.1.
        waves = 1;
        sh->rows = mask_on_device && rows * total > 5120u ? 2 : 1;
    } else if (mask_on_device && sh->policy == DL_POL_STREAM_IN && rows >= 3u && rows <= in_one) {
        // Where sources stream, four wavefronts of up to four rows, all loaded before any is stored (see dl_dispatch_mask_kernel).
        // Eight of two, the counting behind the loads in time : eight of two, loads in a burst : this, and last this with
        // stores as soon as a row is there, three sets in turn: 334 / 430 / 512 per rank of 4 KiB 12.1 / 14.9 / 16.8 : 12.0 / 15.6 /
        // 18.1 : 11.0 / 14.1 / 16.2 : 10.8 / 16.7 / 18.5 us, 170 / 220 / 253 of 8 KiB 12.3 / 15.1 / 16.7 : 12.0 / 15.6 / 17.4 :
        // 11.1 / 14.0 / 15.7 : 10.9 / 15.8 / 16.7, 128 / 192 of 10 KiB (four wavefronts of three, then) 12.1 / 16.4 : 10.7 /
        // 16.4 : 10.8 / 15.6 : 10.4 / 17.5, 112 / 128 of 14 KiB (four of four) 14.1 / 15.7 : 12.7 / 14.1 : 12.7 / 14.2 : 13.5 /
        // 15.0; 450 / 590 of 3 KiB 12.5 / 17.6 before, 11.6 / 16.1 this way.  (Outside this range of sizes, the other way round: 150
        // of 14 KiB 18.7 without the burst, 19.8 with it.  Shorter rows stay with eight of two: 700 of 2 KiB 13.4, 14.0 with four, before the burst lay where it does.)
        waves = 4;
        sh->rows = rows < 4u ? (int)rows : 4;
    } else if (sh->policy != DL_POL_STREAM && rows > 4u && rows <= in_one) {
        // Between: up to four rows of a wavefront in flight together.  Three sets in turn, mask on the host, 192 / 256 per
        // rank of 8 KiB 12.5 / 16.8 : 12.1 / 15.9 us, 128 / 192 of 10 KiB 10.8 / 16.3 : 10.4 / 15.3, 128 of 14 KiB 14.9 : 14.1
        // (one set or sets that fit no cache +-3 %; 384 of 4 KiB 13.3 : 15.9 and 64 of 20 KiB 11.0 : 11.6, which stay).  Mask on the
        // device, less than what streams: 13 rows and more likewise (512 of 14 KiB, which stream, 59.8 : 60.8), and 9 to 12
        // rows, whose five or six wavefronts of two lie badly on four SIMDs, by four of three (384 / 512 of 10 KiB
        // 35.2 / 45.7 : 33.5 / 44.6; 768, in sets that fit no cache, 75.5 : 79.3).
        if (!mask_on_device ? sh->policy == DL_POL_STREAM_IN : rows >= 13u && sh->policy != DL_POL_STREAM_OUT) {
            waves = 4;
            sh->rows = 4;
        } else if (mask_on_device && rows >= 9u && rows <= 12u && bound < (512ull << 20)) {
            waves = 4;
            sh->rows = 3;
        }
    }
    const uint32_t per_wg = waves * (uint32_t)sh->rows;
    sh->grid_x = (uint32_t)((rows + per_wg - 1) / per_wg);
    a->token_waves = (uint32_t)((rows + sh->grid_x * sh->rows - 1) / (sh->grid_x * sh->rows));
    a->wg_tokens = 1;
    while (2u * a->wg_tokens * a->token_waves <= waves) a->wg_tokens *= 2;
    sh->threads = 64u * a->wg_tokens * a->token_waves;
    return DL_OK;
}

// `m` tokens (at most GROUP) of the mask to their group's record; `placed` is carried from group to group.
void pack_group(dispatch_group *g, const uint8_t *mask, uint32_t m, uint32_t (&placed)[DISPATCH_W])
{
    memcpy(g->taken, placed, sizeof placed);
    uint64_t acc = 0;  // bytewise sums of at most 64 words of zeros and ones
    for (uint32_t t = 0; t < m; ++t) {
        uint64_t w;
        memcpy(&w, mask + t * (size_t)DISPATCH_W, sizeof w);
        w |= w >> 4;
        w |= w >> 2;
        w |= w >> 1;
        w &= 0x0101010101010101ull;
        acc += w;
        // the eight low bits into one byte: the multiplication moves bit 8 j to bit 56 + j
        g->ranks[t] = (uint8_t)((w * 0x0102040810204080ull) >> 56);
    }
    memset(g->ranks + m, 0, GROUP - m);
    for (int j = 0; j < DISPATCH_W; ++j) placed[j] += (uint32_t)(acc >> (8 * j)) & 0xFFu;
}

// A few tokens off the grid are lowered on the host (a list in the kernel arguments or a short table): the destinations
// of a row in turn, with their edges, keep one wavefront busy for longer than the host needs for so few items.  Rows of
// 1000 / 14 338 / 16 400 bytes, 1, 4, 16 and 32 tokens per rank: on the host 2.7, 3.1, 5.2 and 7.6 us whatever the
// length, placed on the device 6.7 / 6.9 / 5.2, 7.1 / 7.3 / 5.5, 7.6 / 7.6 / 6.5 and 7.4 / 8.7 / 7.2; at 64 per rank
// 11 to 16 on the host, 7.6 / 11.8 / 12 here.
constexpr uint64_t OFF_GRID_MIN_TOKENS = 256;

// A large request whose mask is in device memory packs the groups first, in a launch of their own, so that the kernel
// that copies need not count: it can then have many small workgroups (see dispatch_setup).  That costs 5 us, and pays from
// the sizes (every token to every rank) below.  One launch : two, sources not in the caches: 14 336 bytes, 700 / 1024 per
// rank (689 / 1008 MiB by this measure) 82 : 86 and 139 : 131 us; 64 KiB, 128 / 256 / 1024 (576 / 1152 / 4608 MiB) 68.5 :
// 69.1, 162 : 148 and 634 : 582; off the grid 16 400 bytes, 128 / 256 / 1024 (144 / 288 / 1153 MiB) 28.3 : 29.7, 49.8 :
// 47.6 and 255 : 194, 14 338 bytes, 512 / 1024 (504 / 1008 MiB) 83.7 : 83.6 and 200 : 188.
constexpr uint64_t PACK_FIRST_BYTES = 900ull << 20;
constexpr uint64_t PACK_FIRST_OFF_GRID_BYTES = 256ull << 20;  // rows longer than a workgroup holds
static_assert((DL_DISPATCH_DEVICE_MAX_TOKENS + GROUP - 1) / GROUP * sizeof(dispatch_group) <= DL_RING_SLOT_BYTES, "groups of the largest request");

// A table cannot be captured into a graph, the kernel arguments can (32 items fit either way).
bool capturing(hipStream_t stream)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (!stream) return false;  // the default stream cannot be captured
    if (hipStreamIsCapturing(stream, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

}  // namespace

int dl_dispatch_on_device(const void *const *in, void *const *out, int W, const uint32_t *tokens, size_t row_bytes,
                          const uint8_t *dest, uint64_t min_tokens, hipStream_t stream, bool *taken)
{
    *taken = false;
    const dl_config &c = g_dl.cfg;
    if (W != DISPATCH_W || !in || !out || !tokens || !dest) return DL_OK;
    if (c.tile_bytes || c.block_threads || c.max_blocks || (c.fan_split != 0 && c.fan_split != DL_TABLE_ROWS_SPLIT)) return DL_OK;
    if (row_bytes == 0) return DL_OK;
    uint64_t total = 0;
    for (int i = 0; i < W; ++i) {
        total += tokens[i];
        if ((tokens[i] && !in[i]) || !out[i]) return DL_OK;  // the host lowering reports what is wrong
    }
    // (a grid has at most 2048 tokens from the kernel arguments or 43 648 through the BAR; from 2^21 on, which would be a
    // thousand launches, a request goes the way of any long list)
    if (total == 0 || total < min_tokens || total >= (1ull << 21)) return DL_OK;

    dispatch_list p;
    dispatch_shape sh;
    int rc = dispatch_setup(in, out, tokens, total, row_bytes, false, &p.a, &sh);
    if (rc != DL_OK) return rc;
    if (!sh.on_grid && total < OFF_GRID_MIN_TOKENS && !(total > 32u && capturing(stream))) return DL_OK;
    const uint64_t groups = (total + GROUP - 1) / GROUP;
    char *pushed = nullptr;
    if (groups > DISPATCH_GROUPS) {
        // too long for the kernel arguments of one launch: all groups through the BAR, if that way is open
        pushed = dl_push_acquire(groups * sizeof(dispatch_group), stream, &rc);
        if (rc != DL_OK) return rc;
    }
    *taken = true;
    uint32_t placed[DISPATCH_W] = {0};
    if (pushed) {
        dispatch_group *slot = (dispatch_group *)pushed;
        for (uint64_t g = 0; g < groups; ++g) {
            dispatch_group one;  // packed here, then written in one go: the slot is write only
            const uint64_t t0 = g * GROUP;
            pack_group(&one, dest + t0 * DISPATCH_W, (uint32_t)(total - t0 < GROUP ? total - t0 : GROUP), placed);
            memcpy(slot + g, &one, sizeof one);
        }
        const dl_pushed ps = dl_push_kernel_args(dl_push_seal(pushed));
        const dim3 grid(sh.grid_x, (uint32_t)((total + p.a.wg_tokens - 1) / p.a.wg_tokens));
        with_instance(sh, [&](auto pol, auto og, auto rows) {
            hipLaunchKernelGGL((dl_dispatch_pushed_kernel<decltype(pol)::value, decltype(og)::value, decltype(rows)::value>), grid, dim3(sh.threads), 0,
                               stream, p.a, (const dispatch_group *)pushed, ps);
        });
        DL_HIP(hipGetLastError());
        return dl_push_commit(stream);
    }
    for (uint64_t g0 = 0; g0 < groups; g0 += DISPATCH_GROUPS) {
        const uint64_t g1 = groups - g0 < DISPATCH_GROUPS ? groups : g0 + DISPATCH_GROUPS;
        for (uint64_t g = g0; g < g1; ++g) {
            const uint64_t t0 = g * GROUP;
            pack_group(&p.group[g - g0], dest + t0 * DISPATCH_W, (uint32_t)(total - t0 < GROUP ? total - t0 : GROUP), placed);
        }
        p.a.token0 = (uint32_t)(g0 * GROUP);
        const uint64_t n = (g1 * GROUP < total ? g1 * GROUP : total) - g0 * GROUP;
        const dim3 grid(sh.grid_x, (uint32_t)((n + p.a.wg_tokens - 1) / p.a.wg_tokens));
        with_instance(sh, [&](auto pol, auto og, auto rows) {
            hipLaunchKernelGGL((dl_dispatch_list_kernel<decltype(pol)::value, decltype(og)::value, decltype(rows)::value>), grid, dim3(sh.threads), 0, stream, p);
        });
        DL_HIP(hipGetLastError());
    }
    return DL_OK;
}

// Token dispatch with the routing mask in device memory (dl_token_dispatch_device): on the caller's stream, and nothing
// of the request but the kernel arguments comes from the host.  One launch, which uses no memory of the library's; or two
// with the groups in its table memory, if the request is large, the stream is not being captured and that memory is free.
extern "C" int dl_token_dispatch_device(const void *const *in, void *const *out, int W, const uint32_t *tokens,
                                        size_t row_bytes, const uint8_t *dest_device, void *stream)
{
    DL_LOCKED;
    if (!g_dl.inited) return DL_ERR_STATE;
    if (dl_device_error_pending()) return DL_ERR_LOST;
    if (W != DISPATCH_W || !in || !out || !tokens) return DL_ERR_INVALID;
    uint64_t total = 0;
    for (int i = 0; i < W; ++i) total += tokens[i];
    if (total == 0 || row_bytes == 0) return DL_OK;
    if (!dest_device || ((uint64_t)dest_device & 7u)) return DL_ERR_INVALID;
    for (int i = 0; i < W; ++i) {
        if ((tokens[i] && !in[i]) || !out[i]) return DL_ERR_INVALID;
    }
    if (total > DL_DISPATCH_DEVICE_MAX_TOKENS) return DL_ERR_CAPACITY;
    dispatch_args a;
    dispatch_shape sh;
    hipStream_t hs = (hipStream_t)stream;
    int rc = dispatch_setup(in, out, tokens, total, row_bytes, true, &a, &sh);
    if (rc != DL_OK) return rc;
    size_t slot;
    dispatch_group *groups = nullptr;
    const uint64_t bound = total * row_bytes * (1u + DISPATCH_W);  // (see dispatch_setup)
    if ((bound >= PACK_FIRST_BYTES || (!sh.on_grid && sh.long_rows && bound >= PACK_FIRST_OFF_GRID_BYTES)) && !capturing(hs))
        groups = (dispatch_group *)dl_scratch_acquire(&slot);
    if (groups) {
        rc = dispatch_setup(in, out, tokens, total, row_bytes, false, &a, &sh);
        if (rc != DL_OK) return rc;
        hipLaunchKernelGGL(dl_dispatch_pack_kernel, dim3((uint32_t)((total + GROUP - 1) / GROUP)), dim3(64 * MAX_WAVES), 0, hs, dest_device,
                           (uint32_t)total, groups);
        DL_HIP(hipGetLastError());
    }
    const dim3 grid(sh.grid_x, (uint32_t)((total + a.wg_tokens - 1) / a.wg_tokens));
    with_instance(sh, [&](auto pol, auto og, auto rows) {
        if (groups)
            hipLaunchKernelGGL((dl_dispatch_packed_kernel<decltype(pol)::value, decltype(og)::value, decltype(rows)::value>), grid,
                               dim3(sh.threads), 0, hs, a, (const dispatch_group *)groups);
        else
            hipLaunchKernelGGL((dl_dispatch_mask_kernel<decltype(pol)::value, decltype(og)::value, decltype(rows)::value>), grid,
                               dim3(sh.threads), 0, hs, a, dest_device);
    });
    DL_HIP(hipGetLastError());
    if (groups) {
        rc = dl_scratch_release(slot, hs);
        if (rc != DL_OK) return rc;
    }
    t_dl_last.mode = DL_MODE_ONESHOT;
    return DL_OK;
}
