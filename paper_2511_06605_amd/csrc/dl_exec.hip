// One-shot execution: a whole lowered copy list in ONE kernel launch (the
// compute-unit analogue of queueing many copies back to back on one engine with
// a single completion, Sec. IV-D, and of spreading one large copy over many
// engines, Sec. IV-A).
//
// Short lists travel by value in the kernel-argument segment, so the device
// needs no extra memory round trip to find its work: workgroup b finds its
// (item, tile) from an inclusive prefix sum of tile counts.  Long lists of equal
// plain copies travel there as offsets.  Other long lists are cut
// into one-tile entries on the host and become a table, workgroup b taking
// entry b: written straight into device memory through the BAR where that is
// possible (see push_acquire), else into a pinned host ring (and copied to
// device memory first when there are many entries).
#include "dl_device.h"
#include "dl_internal.h"

#include <immintrin.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

// ------------------------------------------------------------------- kernels

// Row path only (see dl_run_rows).  A kernel of its own: sharing one kernel with
// the general path cost 5 % of the all-gather rate through its register count.
// ON_GRID: see dl_rows_body.
template <class Item, int NMAX, int POL, bool ON_GRID>
__global__ void __launch_bounds__(512) dl_exec_rows_kernel(const dl_klist<Item, NMAX> p)
{
    dl_run_rows<POL, ON_GRID>(p, blockIdx.x);
}

// Row path over a list too long for the scalar compares of dl_find_item (the 64 chunks of an all-to-all between
// eight ranks): a two-dimensional grid, blockIdx.y the item, blockIdx.x the tile within it, so nothing is
// searched and nothing divided.  The grid is as wide as the longest item; a workgroup beyond its item's last
// row leaves at once (the host takes this path only while few workgroups are wasted that way).  Consecutive
// workgroups walk along one item, so the chip-wide stream of addresses stays sequential (EIGHTHS: see dl_eighths_tile).
template <class Item, int NMAX, int POL, bool ON_GRID, bool EIGHTHS = false>
__global__ void __launch_bounds__(512) dl_exec_rows2d_kernel(const dl_klist<Item, NMAX> p)
{
    const uint32_t tile = EIGHTHS ? dl_eighths_tile(blockIdx.x, gridDim.x) : blockIdx.x;
    dl_rows_body<POL, ON_GRID>(p.item[blockIdx.y], tile, p.wpg_log2, p.split_log2);
}

// Large copies with several destinations, written two destinations at a time (see dl_pair_body).
template <int NMAX, int POL, bool ON_GRID>
__global__ void __launch_bounds__(64) dl_exec_pairs_kernel(const dl_klist<dl_fused_item, NMAX> p)
{
    uint32_t first;
    const uint32_t d = dl_find_item(p, blockIdx.x, &first);
    if (d < p.n) dl_pair_body<POL, ON_GRID>(p.item[d], blockIdx.x - first);
}

// Entry i of a table that the host wrote into device memory through the BAR just before the launch.  A line
// of the table that used this memory before may still sit in a cache, so the entry is read past every cache,
// once per workgroup (8 bytes per lane), and handed on through LDS; before that, one lane has seen the slot's
// stamp.  Call with the whole workgroup.  Null if the stamp never came (reported by the caller).
template <class Item>
__device__ __forceinline__ const Item *dl_pushed_entry(const Item *items, uint32_t i, const dl_pushed &ps)
{
    constexpr uint32_t WORDS = sizeof(Item) / 8;
    static_assert(sizeof(Item) % 8 == 0 && WORDS < 64, "one 8-byte load per lane of the first wavefront");
    __shared__ uint64_t raw[WORDS];
    __shared__ uint32_t sealed;
    if (threadIdx.x == 0) sealed = dl_pushed_sealed(items, ps) ? 1u : 0u;
    __syncthreads();
    if (!sealed) return nullptr;
    if (threadIdx.x < WORDS) raw[threadIdx.x] = dl_ld<DL_POL_COHERENT>(dl_global<uint64_t>(items + i) + threadIdx.x);
    __syncthreads();
    return reinterpret_cast<const Item *>(raw);
}

// Row path over a table of equally sized items in device memory (long lists: thousands of token
// rows, hundreds of cache blocks) on a two-dimensional grid: blockIdx.y is the item (at most DL_UROWS_MAX_ITEMS,
// the grid's limit in that dimension), which every workgroup of that item finds in the scalar cache, blockIdx.x
// the tile within it; nothing is divided.  PUSHED: see dl_pushed_entry.
template <class Item, int POL, bool PUSHED, bool ON_GRID>
__global__ void __launch_bounds__(512) dl_exec_urows_kernel(const Item *__restrict__ items, uint32_t wpg_log2,
                                                            uint32_t split_log2, const dl_pushed ps)
{
    const uint32_t d = blockIdx.y;
    if constexpr (PUSHED) {
        const Item *it = dl_pushed_entry(items, d, ps);
        if (it)
            dl_rows_body<POL, ON_GRID>(*it, blockIdx.x, wpg_log2, split_log2);
        else if (threadIdx.x == 0)
            dl_pushed_report_lost(ps);  // nothing copied by this workgroup; the host hears of it
    } else
        dl_rows_body<POL, ON_GRID>(items[d], blockIdx.x, wpg_log2, split_log2);
}

// Row path over equally long copies given by offsets in the kernel arguments (cache blocks moved between two pools):
// blockIdx.y the item, blockIdx.x the tile within it.  Nothing is fetched through memory that the host has just
// written, so the two round trips in front of every row of a pushed table (stamp, entry) are gone: 256 copies of 64 KiB
// 7.4 us of kernel, now 6.2 (10.4 -> 9.8 us a call); of 256 KiB 28.5 -> 21.6 us, of 1 MiB 97.3 -> 85.7 us, where one-wavefront
// workgroups count as well.
template <class Item, int NMAX, int POL, bool ON_GRID, bool EIGHTHS = false>
__global__ void __launch_bounds__(512) dl_exec_offsets_kernel(const dl_offset_list<NMAX> p)
{
    const uint32_t d = blockIdx.y;
    Item it;
    it.src = p.src + ((uint64_t)p.at[d].src << p.unit_log2);
    it.dst = p.dst + ((uint64_t)p.at[d].dst << p.unit_log2);
    it.bytes = p.bytes;
    dl_rows_body<POL, ON_GRID>(it, EIGHTHS ? dl_eighths_tile(blockIdx.x, gridDim.x) : blockIdx.x, p.wpg_log2, 0u);
}

// General path: any tile size, one workgroup per tile.
template <class Item, int NMAX, int POL>
__global__ void __launch_bounds__(512) dl_exec_list_kernel(const dl_klist<Item, NMAX> p)
{
    dl_run_tile<POL>(p, blockIdx.x);
}

// Same, with a capped grid: workgroup b takes tiles b, b + grid, b + 2 grid, ...
template <class Item, int NMAX, int POL>
__global__ void __launch_bounds__(512) dl_exec_list_strided_kernel(const dl_klist<Item, NMAX> p)
{
    const uint32_t total = p.tile_end[p.n - 1];
    for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) dl_run_tile<POL>(p, b);
}

template <class Item, int POL, bool PUSHED = false>
__global__ void __launch_bounds__(512) dl_exec_table_kernel(const Item *__restrict__ items, uint32_t n, uint32_t split,
                                                            const dl_pushed ps)
{
    const uint32_t b = blockIdx.x;
    if (b >= n) return;
    if constexpr (PUSHED) {
        const Item *pushed = dl_pushed_entry(items, b, ps);
        if (!pushed) {
            if (threadIdx.x == 0) dl_pushed_report_lost(ps);  // nothing copied by this workgroup; the host hears of it
            return;
        }
        const Item it = *pushed;
        dl_run_entry<POL>(it, split);
    } else {
        const Item it = items[b];
        dl_run_entry<POL>(it, split);
    }
}

// ------------------------------------------------------------ armed kernels
//
// The compute-unit analogue of a poll command queued in front of the copies
// (Sec. IV-E): the kernel is enqueued ahead of time, its workgroups wait until
// the doorbell word (in device memory that the host writes through the BAR, else
// in host-coherent memory) reaches their ticket, then copy.
// No workgroup ever waits for another one to make progress, and every wait is
// bounded by a wall-clock limit, so every wave leaves the kernel.

enum : uint32_t { DL_GO_WAIT = 0, DL_GO_RUN = 1, DL_GO_SKIP = 2 };

// First thing in a kernel that may count its workgroups in: the counters that the slot's next request that counts will
// use, one lane each.  The stores are in flight beside the wait and the copy.
__device__ __forceinline__ void dl_arm_clear(const dl_arm &a)
{
    static_assert(DL_ARM_GROUPS < 64, "one lane per counter");
    if (a.arrive_clear && blockIdx.x == 0 && threadIdx.x <= DL_ARM_GROUPS)
        __hip_atomic_store((uint32_t *)((char *)a.arrive_clear + threadIdx.x * DL_ARM_STRIDE), 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// Tells the host that a kernel that waits is on the device.
__device__ __forceinline__ void dl_arm_resident(const dl_arm &a)
{
    __hip_atomic_store(a.armed, a.ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Phase stamps of a request that waits for no doorbell.
__device__ __forceinline__ void dl_arm_stamp_begin(const dl_arm &a)
{
    if (a.trace_host && blockIdx.x == 0 && threadIdx.x == 0) {
        const uint64_t t = (uint64_t)wall_clock64();
        __hip_atomic_store(a.trace_host, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(a.trace_host + 1, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// One thread polls the doorbell (system-scope loads past every cache: device memory, or host memory over the link) until
// it has been rung for this ticket, the request is cancelled or the limit runs out.  t0: when the kernel began to wait.
__device__ __forceinline__ uint32_t dl_arm_poll(const dl_arm &a, uint64_t t0, bool pause)
{
    for (uint32_t spins = 1;; ++spins) {
        // doorbell and cancel word sit side by side in one aligned 16 bytes: one read over the link
        // (each is an aligned 8-byte word that the host writes with one store, so neither can tear)
        const dl_u32x4 w = dl_ld<DL_POL_COHERENT>(dl_global<dl_u32x4>(a.bell));
        const uint64_t bell = (uint64_t)w.x | ((uint64_t)w.y << 32);
        const uint64_t cancel = (uint64_t)w.z | ((uint64_t)w.w << 32);
        if (cancel >= a.ticket) return DL_GO_SKIP;
        if (bell >= a.ticket) return DL_GO_RUN;
        if ((spins & 3u) == 0 && (uint64_t)wall_clock64() - t0 > a.limit_ticks) return DL_GO_SKIP;
        if (spins >= a.max_spins) return DL_GO_SKIP;
        if (pause) __builtin_amdgcn_s_sleep(8);
    }
}

__device__ __forceinline__ void dl_arm_stamp(const dl_arm &a, int which)
{
    if (a.trace_host && blockIdx.x == 0)
        __hip_atomic_store(a.trace_host + which, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Returns DL_GO_RUN once the doorbell has been rung for this ticket, DL_GO_SKIP
// if the request was cancelled or the limit ran out.  Uniform over the workgroup.
__device__ __forceinline__ uint32_t dl_arm_wait(const dl_arm &a)
{
    __shared__ uint32_t s_go;
    dl_arm_clear(a);
    if (a.nowait && a.gated) {
        // uniform over the grid: the waiting was done by the gate kernel that ran before this one on the stream
        // (see dl_arm_gate_kernel); what it decided lies in the slot's first flag
        if (threadIdx.x == 0) {
            const uint64_t g = __hip_atomic_load(a.go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_go = (g >> 2) == a.ticket ? (uint32_t)(g & 3u) : (uint32_t)DL_GO_SKIP;
            if (s_go == DL_GO_RUN) dl_arm_stamp(a, 1);
        }
        __syncthreads();
        return s_go;
    }
    if (a.nowait) {  // uniform over the grid: started without a doorbell
        dl_arm_stamp_begin(a);
        return DL_GO_RUN;
    }
    if (threadIdx.x == 0) {
        uint32_t go = DL_GO_SKIP;
        const uint64_t t0 = wall_clock64();
        if (blockIdx.x == 0) dl_arm_resident(a);  // before the wait: off the critical path
        if (a.direct || blockIdx.x == 0) {
            go = dl_arm_poll(a, t0, blockIdx.x && !a.direct);
            if (go == DL_GO_RUN) dl_arm_stamp(a, 0);
            if (!a.direct) {
                // pass the word on: one flag per group of workgroups, each in its own cache line
                // (the flag carries everything the others need, so it is not ordered against anything)
                const uint32_t groups = gridDim.x < DL_ARM_GROUPS ? gridDim.x : DL_ARM_GROUPS;
                for (uint32_t g = 0; g < groups; ++g)
                    __hip_atomic_store((uint64_t *)((char *)a.go + g * DL_ARM_STRIDE), (a.ticket << 2) | go,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            // wait for workgroup 0 to pass the word on through device memory
            const uint64_t *flag = (const uint64_t *)((const char *)a.go + (blockIdx.x % DL_ARM_GROUPS) * DL_ARM_STRIDE);
            for (uint32_t spins = 1;; ++spins) {
                const uint64_t g = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((g >> 2) == a.ticket) {
                    go = (uint32_t)(g & 3u);
                    break;
                }
                __builtin_amdgcn_s_sleep(8);
                if ((spins & 15u) == 0 && (uint64_t)wall_clock64() - t0 > a.limit_ticks + a.margin_ticks) break;
                if (spins >= a.max_spins) break;
            }
        }
        if (go == DL_GO_RUN) dl_arm_stamp(a, 1);  // the polling workgroup is the first to begin its copy
        s_go = go;
    }
    __syncthreads();
    // No cache invalidate here: the copy that follows loads at system scope (DL_POL_COHERENT), so
    // it sees everything that was written before the doorbell was rung.
    return s_go;
}

// Count this workgroup in; the last one to arrive publishes the completion word.
// Arrivals are counted per group first (a counter per cache line), and the last
// of each group is counted at the top, so no counter sees more than
// grid / DL_ARM_GROUPS + DL_ARM_GROUPS updates.  The low 16 bits of a counter
// count arrivals, the high bits count workgroups that skipped the copy.
//
// No cache write-back anywhere: the copy stored at system scope, so once every
// wavefront has drained its memory counter the workgroup's bytes are visible to
// the host and to every later kernel, and relaxed counters suffice.  (With
// ordinary stores each workgroup had to write the L2 back before counting
// itself in; that serialised per XCD and cost ~0.5 us per workgroup.)
__device__ __forceinline__ void dl_arm_report(const dl_arm &a, uint32_t go)
{
    if (a.own_word) {
        // a small grid: the host waits for one word per workgroup, no count in between
        __hip_atomic_store(a.done + blockIdx.x, a.ticket | (go == DL_GO_RUN ? 0ull : DL_DONE_SKIPPED), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    {
        const uint32_t grid = gridDim.x;
        const bool flat = grid <= DL_ARM_FLAT_MAX;  // few enough to count at one word without queueing there
        const uint32_t groups = flat ? grid : DL_ARM_GROUPS;
        const uint32_t g = blockIdx.x % DL_ARM_GROUPS;
        const uint32_t gsize = (grid - g + DL_ARM_GROUPS - 1) / DL_ARM_GROUPS;
        uint32_t *gcount = (uint32_t *)((char *)a.arrive + g * DL_ARM_STRIDE);
        uint32_t *top = (uint32_t *)((char *)a.arrive + DL_ARM_GROUPS * DL_ARM_STRIDE);
        // this workgroup's stores have drained; the workgroup that turns out to be the last of all reports
        // its own reading as the end of the last copy (no extra traffic for the others)
        const uint64_t t_end = a.trace_host ? (uint64_t)wall_clock64() : 0ull;
        uint32_t add = 1u + (go == DL_GO_RUN ? 0u : 0x10000u);
        uint32_t old;
        if (!flat) {
            old = __hip_atomic_fetch_add(gcount, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((old & 0xFFFFu) != gsize - 1u) return;
            // last of the group: carry the result to the top
            add = 1u + (((old >> 16) + (add >> 16)) << 16);
        }
        // a small grid is counted at the top directly
        old = __hip_atomic_fetch_add(top, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((old & 0xFFFFu) != groups - 1u) return;
        // last of all
        // The counters stay as they are: the slot's next request counts on the other set and clears this one
        // (see dl_arm).  Nothing is in flight from this wavefront here except, when tracing, the stamps, which
        // must have landed before the completion word.
        const uint32_t skipped = (old >> 16) + (add >> 16);
        if (a.trace_host) {
            __hip_atomic_store(a.trace_host + 2, t_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(a.trace_host + 3, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            dl_drain_stores();
        }
        __hip_atomic_store(a.done, a.ticket | (skipped ? DL_DONE_SKIPPED : 0ull), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__device__ __forceinline__ void dl_arm_finish(const dl_arm &a, uint32_t go)
{
    dl_drain_stores();
    __syncthreads();
    if (threadIdx.x == 0) dl_arm_report(a, go);
}

// Gate of a large prelaunched request.  A grid that waits for a doorbell must stay small (see armed_grid), and a
// small grid is what bounds a large copy.  So the waiting is done by this kernel, one workgroup, and the copy by
// an ordinary signal-style kernel with a full grid that is enqueued behind it on the same stream: it starts when
// this one ends, reads what this one decided, and copies or reports that the request gave up.  One more kernel
// start (0.5-1.5 us measured) on the critical path, which pays from about 256 MiB moved; and while the request waits it
// holds one workgroup instead of one on every other compute unit.
__global__ void __launch_bounds__(64) dl_arm_gate_kernel(const dl_arm a)
{
    const uint32_t go = dl_arm_wait(a);
    if (threadIdx.x == 0)
        __hip_atomic_store(a.go, (a.ticket << 2) | (uint64_t)go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A signalled request on the row path: no doorbell, a workgroup per tile, then the report.  A kernel of its own, because what
// it takes beyond a one-shot kernel's time is instruction fetch and round trips: nothing of the waiting kernels' code is in
// the way, and the loads are ordinary ones (whoever wrote the sources did so before the launch).
template <class Item, int NMAX, bool ON_GRID>
__global__ void __launch_bounds__(512) dl_signal_rows_kernel(const dl_klist<Item, NMAX> p, const dl_arm a)
{
    dl_arm_clear(a);
    dl_arm_stamp_begin(a);
    dl_run_rows<DL_POL_WT, ON_GRID>(p, blockIdx.x);
    dl_arm_finish(a, DL_GO_RUN);
}

// Completion of a large signalled request: the copy is an ordinary one-shot kernel (whose stores are at system scope), and this
// one, behind it on the stream, reports.
__global__ void __launch_bounds__(64) dl_signal_done_kernel(uint64_t *done, uint64_t ticket)
{
    if (threadIdx.x == 0) __hip_atomic_store(done, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A waiting request of at most one tile per workgroup, each of which polls the doorbell itself.  Whatever the copy needs is
// worked out before the wait, so that behind it there are a load, the stores and the report, in few instructions: what
// counts there is instruction fetch and round trips.
template <class Item, int NMAX, bool ON_GRID>
__global__ void __launch_bounds__(1024) dl_armed_rows_kernel(const dl_klist<Item, NMAX> p, const dl_arm a)
{
    constexpr int K = std::is_same<Item, dl_plain_item>::value ? 1 : DL_FAN;
    __shared__ uint32_t s_go;
    const uint64_t t0 = wall_clock64();
    dl_arm_clear(a);
    if (blockIdx.x == 0 && threadIdx.x == 0) dl_arm_resident(a);
    uint32_t first;
    const uint32_t d = dl_find_item(p, blockIdx.x, &first);  // (< p.n: the grid is as long as the list has tiles)
    const Item &it = p.item[d];
    const char *const src = it.src;
    const uint64_t bytes = it.bytes;
    char *dst[K];
#pragma unroll
    for (int q = 0; q < K; ++q) dst[q] = (char *)dl_item_dst(it, (uint32_t)q);  // filled from the front, the rest null
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wl = p.wpg_log2;
    const uint64_t row = ((uint64_t)(blockIdx.x - first) << wl) + (wave & ((1u << wl) - 1u));
    const uint32_t shift = ON_GRID ? 0u : dl_item_shift(it);
    const uint32_t kind = ON_GRID ? (uint32_t)DL_ROW_PLAIN : dl_row_kind(dl_item_ragged(it), shift, bytes, row);
    const uint64_t byte = ((row << 10) - shift) + (lane << 4);
    const bool whole = dl_lane_whole(byte, bytes, kind);
    asm volatile("" ::"s"(src), "s"(dst[0]), "s"(dst[K - 1]), "v"(byte));
    if (threadIdx.x == 0) {
        const uint32_t go = dl_arm_poll(a, t0, false);
        if (go == DL_GO_RUN) {
            dl_arm_stamp(a, 0);
            dl_arm_stamp(a, 1);
        }
        s_go = go;
    }
    __syncthreads();
    const uint32_t go = s_go;
    if (go == DL_GO_RUN) {
        if (kind == DL_ROW_EDGE)
            dl_row_edges(shift, bytes, row, lane, [&](uint64_t i) {
                const uint8_t x = dl_ld<DL_POL_COHERENT>(dl_global<uint8_t>(src) + i);
#pragma unroll 1
                for (int q = 0; q < K; ++q) {
                    char *dq = (char *)dl_item_dst(it, (uint32_t)q);
                    if (!dq) break;
                    dl_st<DL_POL_COHERENT>(dl_global<uint8_t>(dq) + i, x);
                }
            });
        if (whole) {
            const dl_u32x4 v = dl_ld16<DL_POL_COHERENT>(src + byte);
#pragma unroll
            for (int q = 0; q < K; ++q) {
                if (!dst[q]) break;
                dl_st16<DL_POL_COHERENT>(dst[q] + byte, v);
            }
        }
    }
    dl_arm_finish(a, go);
}

// The same for a request of more tiles than the waiting grid has workgroups: R tiles a pass, the first pass's worked out
// before the wait.  R is two while two passes are enough for sixteen wavefronts a workgroup, one pass for eight, else four
// (all-gather, trigger to done and the call, sixteen wavefronts, two : four, 608 / 640 / 768 KiB per rank over eight ranks, 2.4 to 3 tiles a
// workgroup, 21.5 / 21.4 / 21.9 : 21.7 / 21.7 / 22.3 us, 1 MiB over five 19.1 : 19.3 and over eight, 4 tiles, 25.0 : 26.2; 2 MiB 56.8 : 47.7).
template <class Item, int NMAX, int R>
__global__ void __launch_bounds__(1024) dl_armed_passes_kernel(const dl_klist<Item, NMAX> p, const dl_arm a)
{
    __shared__ uint32_t s_go;
    const uint64_t t0 = wall_clock64();
    dl_arm_clear(a);
    if (blockIdx.x == 0 && threadIdx.x == 0) dl_arm_resident(a);
    const uint32_t grid = gridDim.x, total = p.tile_end[p.n - 1];
    dl_coherent_rows<R, Item, NMAX> rows;
    rows.prepare(p, blockIdx.x, grid, total, a.go);
    {
        uint64_t touched = 0;  // so that the destinations are in the scalar cache behind the wait
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (rows.d[r] < p.n) touched += (uint64_t)dl_item_dst(p.item[rows.d[r]], 0) + (uint64_t)dl_item_dst(p.item[rows.d[r]], DL_FAN - 1);
        asm volatile("" ::"s"(touched));
    }
    if (threadIdx.x == 0) {
        const uint32_t go = dl_arm_poll(a, t0, false);
        if (go == DL_GO_RUN) {
            dl_arm_stamp(a, 0);
            dl_arm_stamp(a, 1);
        }
        s_go = go;
    }
    __syncthreads();
    const uint32_t go = s_go;
    if (go == DL_GO_RUN) {
        rows.run(p);
        for (uint32_t b = blockIdx.x + R * grid; b < total; b += R * grid) dl_run_rows_coherent<R>(p, b, grid, total, a.go);
    }
    dl_arm_finish(a, go);
}

template <class Item, int NMAX, bool ROWS>
__global__ void __launch_bounds__(512) dl_armed_list_kernel(const dl_klist<Item, NMAX> p, const dl_arm a)
{
    {
        // Before the wait: read what the workgroup's first tile will need from the list, so that after the
        // doorbell those scalar loads hit the scalar cache instead of going to memory one after the other.
        uint32_t first;
        const uint32_t d = dl_find_item(p, blockIdx.x, &first);
        uint64_t touched = first + p.n + p.tile_end[p.n - 1];
        if (d < p.n) {
            const Item &it = p.item[d];
            touched += (uint64_t)it.src + it.bytes + (uint64_t)dl_item_dst(it, 0) + (uint64_t)dl_item_dst(it, DL_FAN - 1);
        }
        asm volatile("" ::"s"(touched));
    }
    const uint32_t go = dl_arm_wait(a);
    if (go == DL_GO_RUN) {
        const uint32_t total = p.tile_end[p.n - 1];
        if constexpr (ROWS && !std::is_same<Item, dl_swap_item>::value) {
            // A grid that makes several passes (it is capped while it waits) keeps four rows in flight per
            // wavefront, or two: a coherent load takes a microsecond or two, and one per pass left the memory idle.
            const uint32_t grid = gridDim.x;
            if (total <= grid)
                dl_run_rows<DL_POL_COHERENT>(p, blockIdx.x);
            else if (p.split_log2 != 0)  // (a forced shape: the several-rows form knows one sub-group only)
                for (uint32_t b = blockIdx.x; b < total; b += grid) dl_run_rows<DL_POL_COHERENT>(p, b);
            else if (total <= 2u * grid)
                dl_run_rows_coherent<2>(p, blockIdx.x, grid, total, a.go);
            else
                for (uint32_t b = blockIdx.x; b < total; b += 4u * grid) dl_run_rows_coherent<4>(p, b, grid, total, a.go);
        } else {
            for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {
                if constexpr (ROWS)
                    dl_run_rows<DL_POL_COHERENT>(p, b);
                else
                    dl_run_tile<DL_POL_COHERENT>(p, b);
            }
        }
    }
    dl_arm_finish(a, go);
}

// What a standby executor reads once its doorbell has rung.  The two copies of the ticket and the activation
// number let the executor refuse a record that is not the one its doorbell announced.
struct dl_standby_rec {
    uint64_t ticket_front;
    uint64_t activation;  // which arming of this pool slot the record is for (the executor's doorbell value)
    uint64_t *done;       // the request's completion words (host-coherent): one per tile up to DL_DONE_WORDS tiles, else one
    uint64_t arrivals;    // written as 0; requests of more than DL_DONE_WORDS tiles count their workgroups in here
    uint64_t plain;       // 1: `copies` holds the request (up to 64 plain copies); 0: `list` (up to 8 read-once/write-k items)
    union {
        dl_klist<dl_fused_item, 8> list;
        dl_klist<dl_plain_item, 64> copies;
    };
    uint64_t ticket_back;
};
static_assert(sizeof(dl_standby_rec) <= DL_STANDBY_REC_BYTES && sizeof(dl_standby_rec) % 8 == 0, "record size");
static_assert(offsetof(dl_standby_rec, list.tile_end) == offsetof(dl_standby_rec, copies.tile_end) &&
                  offsetof(dl_standby_rec, list.n) == offsetof(dl_standby_rec, copies.n),
              "the two kinds of list start alike");

// Standby executor: a generic armed kernel (see dl_internal.h).  Its doorbell is its pool slot's, its "ticket"
// the slot's activation number; the request's own ticket and completion words come with the record.  Workgroup b
// copies tile b of the request; workgroups beyond its last tile have nothing to do and nothing to report.
__global__ void __launch_bounds__(DL_STANDBY_THREADS) dl_standby_kernel(dl_standby_rec *rec_mem, const dl_arm a)
{
    constexpr uint32_t VEC = (uint32_t)((sizeof(dl_standby_rec) + 15) / 16);
    static_assert(VEC <= DL_STANDBY_THREADS, "one 16-byte load per thread fetches the record");
    __shared__ dl_u32x4 raw[VEC];
    if (dl_arm_wait(a) != DL_GO_RUN) return;  // cancelled or never used: no request, nothing to report
    // the record was complete before the doorbell was rung; these loads go to where it lies (device or host
    // memory), past every cache
    if (threadIdx.x < VEC) raw[threadIdx.x] = dl_ld<DL_POL_COHERENT>(dl_global<dl_u32x4>(rec_mem) + threadIdx.x);
    __syncthreads();
    const dl_standby_rec &rec = *reinterpret_cast<const dl_standby_rec *>(raw);
    // n, tile_bytes, split and tile_end[] sit at the same offsets in both kinds of list
    const uint32_t n_max = rec.plain ? 64u : 8u;
    const bool ok = rec.ticket_front != 0 && rec.ticket_front == rec.ticket_back && rec.activation == a.ticket &&
                    rec.done != nullptr && rec.list.n >= 1 && rec.list.n <= n_max && rec.list.tile_bytes == DL_STANDBY_TILE &&
                    rec.list.split == 1 && rec.copies.tile_end[rec.list.n - 1] <= gridDim.x;
    if (!ok) return;  // not the announced record: touch nothing (the host's wait for the request times out)
    const uint32_t tiles = rec.copies.tile_end[rec.list.n - 1];
    if (blockIdx.x >= tiles) return;
    if (rec.plain)
        dl_run_rows<DL_POL_COHERENT>(rec.copies, blockIdx.x);
    else
        dl_run_rows<DL_POL_COHERENT>(rec.list, blockIdx.x);
    // the copy stored at system scope: once the memory counters have drained, the bytes are where everybody sees them
    dl_drain_stores();
    __syncthreads();
    if (threadIdx.x != 0) return;
    if (tiles <= DL_DONE_WORDS) {
        // the host waits for one word per tile, no count in between
        __hip_atomic_store(rec.done + blockIdx.x, rec.ticket_front, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else {
        // count in at the record (device memory: the host sends such requests only there); the last one reports
        const uint64_t before = __hip_atomic_fetch_add(&rec_mem->arrivals, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == tiles - 1u)
            __hip_atomic_store(rec.done, rec.ticket_front, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Entry i of a table written through the BAR (see dl_pushed_entry), read by every lane for itself: all lanes
// load the same 8 bytes, which costs one request per wavefront, and no barrier.  For kernels that walk a table.
// *sealed: the slot's stamp has been seen (looked for here, before the entry is read, unless an earlier call
// saw it already: once the stamp is there the whole table is); if it is not, the entry is not to be used.
template <class Item>
__device__ __forceinline__ Item dl_pushed_entry_per_lane(const Item *items, uint32_t i, const dl_pushed &ps, bool *sealed)
{
    static_assert(sizeof(Item) % 8 == 0, "whole 8-byte words");
    union {
        Item it;
        uint64_t w[sizeof(Item) / 8];
    } u;
    if (!*sealed) *sealed = dl_uniform64(dl_pushed_sealed(items, ps) ? 1ull : 0ull) != 0;
#pragma unroll
    for (uint32_t q = 0; q < sizeof(Item) / 8; ++q) {
        const uint64_t v = *sealed ? dl_ld<DL_POL_COHERENT>(dl_global<uint64_t>(items + i) + q) : 0ull;
        u.w[q] = dl_uniform64(v);  // the same in every lane: keep it in scalar registers
    }
    return u.it;
}

// PUSHED: the table was written through the BAR when the request was armed; the workgroup's first entry is
// fetched before the wait.
template <class Item, bool PUSHED = false>
__global__ void __launch_bounds__(512) dl_armed_table_kernel(const Item *__restrict__ items, uint32_t n, uint32_t split,
                                                             const dl_pushed ps, const dl_arm a)
{
    if constexpr (PUSHED) {
        Item it{};
        bool sealed = blockIdx.x >= n;  // looked for with the first entry; once the stamp has been seen the whole table is there
        if (blockIdx.x < n) it = dl_pushed_entry_per_lane(items, blockIdx.x, ps, &sealed);
        uint32_t go = dl_arm_wait(a);
        if (!sealed && go == DL_GO_RUN) go = DL_GO_SKIP;  // reported like a request that gave up
        if (go == DL_GO_RUN) {
            for (uint32_t b = blockIdx.x; b < n; b += gridDim.x) {
                if (b != blockIdx.x) it = dl_pushed_entry_per_lane(items, b, ps, &sealed);
                dl_run_entry<DL_POL_COHERENT>(it, split);
            }
        }
        dl_arm_finish(a, go);
    } else {
        const uint32_t go = dl_arm_wait(a);
        if (go == DL_GO_RUN) {
            for (uint32_t b = blockIdx.x; b < n; b += gridDim.x) {
                const Item it = items[b];
                dl_run_entry<DL_POL_COHERENT>(it, split);
            }
        }
        dl_arm_finish(a, go);
    }
}

// ---------------------------------------------------------------- host side

namespace {

constexpr int NMAX_SMALL = 8;
template <class Item> struct list_cap;
template <> struct list_cap<dl_plain_item> { static constexpr int big = 64; };
template <> struct list_cap<dl_swap_item> { static constexpr int big = 64; };
template <> struct list_cap<dl_fused_item> { static constexpr int big = 32; };

constexpr uint32_t DL_UROWS_MAX_ITEMS = 65535;    // a grid's second dimension goes no further
constexpr uint64_t TABLE_ENTRIES_TARGET = 8192;  // table kernels: aim for at most this many one-tile entries
constexpr uint64_t FAN_WAVE_MIN_BYTES = 3ull << 20;         // bytes moved above which a copy with several destinations takes one wavefront per row
constexpr uint64_t UNIFORM_ROWS_MIN_BYTES = 4ull << 20;  // source bytes from which a uniform long list takes the row kernel
constexpr uint64_t UNIFORM_ROWS_STAGE_BYTES = 768ull << 20;  // bytes moved (read + written) from which its table is staged even where it could be pushed
constexpr uint64_t STREAM_BOTH_MIN_BYTES = 512ull << 20;  // bytes moved from which lists of plain copies outside the row path stream both sides
constexpr uint64_t OFF_GRID_MIN_BYTES = 24ull << 20;  // bytes moved from which plain copies off the grid keep rows next to each other together
constexpr uint32_t SIGNAL_MAX_BLOCKS = 32768;  // the arrival counters keep 16 bits for the count
constexpr uint64_t SIGNAL_DONE_MIN_BYTES = 12ull << 20;  // bytes moved from which a signalled request is a one-shot kernel and one that reports
constexpr uint64_t RAGGED_GRID = 768;  // workgroups of a two-dimensional grid that may be mostly idle
constexpr uint64_t OFFSETS_MIN_BYTES = 64ull << 20;  // bytes moved per launch where a long uniform list takes several instead of a table
constexpr uint64_t ARMED_ROWS_MAX_BYTES = 32ull << 20;  // bytes moved up to which an armed kernel that does not wait takes the row path for more than eight items
constexpr size_t TABLE_STAGE_MIN = 512;          // tables at least this long are staged in device memory first
constexpr size_t RING_SLOTS = 4;
constexpr size_t RING_SLOT_BYTES = DL_RING_SLOT_BYTES;

constexpr size_t PUSH_SLOT_BYTES = DL_PUSH_SLOT_BYTES;        // a slot of the tables written through the BAR
constexpr size_t PUSH_PAYLOAD_BYTES = DL_PUSH_PAYLOAD_BYTES;  // the longest such table
constexpr size_t PUSH_SLOTS = 64, PUSH_BATCH = PUSH_SLOTS / 2;

struct ring_t {
    char *base = nullptr;  // pinned host memory: the host writes tables here
    char *dev = nullptr;   // device memory of the same shape: long tables are staged here before they are used
    // Tables written through the BAR (see push_acquire): PUSH_SLOTS slots of device memory that the host can
    // store into, used in turn.  Before a slot is used again the kernel that read its table must have ended:
    // cover[s] names the slot whose event was recorded behind that kernel.  On a stream that cannot go away
    // between calls (the default stream, the library's own) the launches of up to PUSH_BATCH calls in a row
    // share one event, recorded behind the last of them; on a caller's stream every launch gets its own, while
    // the handle is known to be good.
    char *push = nullptr;
    size_t push_next = 0;                 // slot that the next table takes
    hipEvent_t push_ev[PUSH_SLOTS]{};
    int push_cover[PUSH_SLOTS]{};         // -1: never used, or used in the batch that is still open
    bool push_used[PUSH_SLOTS]{};
    uint64_t push_armed[PUSH_SLOTS]{};    // ticket of the armed (prelaunch mode) request whose table is in the slot, or 0
    size_t batch_first = 0, batch_len = 0;  // the open batch: slots batch_first .. batch_first + batch_len - 1 (mod PUSH_SLOTS)
    hipStream_t batch_stream = nullptr;
    hipStream_t own_stream = nullptr;     // the library's stream for armed requests, while it exists
    // the pinned ring: an event per slot, recorded behind the kernel that reads it
    hipEvent_t ev[RING_SLOTS]{};
    bool used[RING_SLOTS]{};
    uint64_t armed[RING_SLOTS]{};         // ticket of the armed (prelaunch mode) request whose table is in the slot, or 0
    size_t next = 0;
} g_ring;

// The item's first destination stands on a DL_CUT boundary, its length is a multiple of 16 and its source one of 4.
template <class Item>
inline bool item_on_grid(const Item &it)
{
    return dl_item_shift(it) == 0 && (it.bytes & 15u) == 0 && ((uint64_t)it.src & 3u) == 0;
}

template <class Item>
bool all_on_grid(const Item *items, size_t n)
{
    for (size_t i = 0; i < n; ++i)
        if (!item_on_grid(items[i])) return false;
    return true;
}

inline uint32_t log2u(uint32_t v)
{
    uint32_t l = 0;
    while ((2u << l) <= v) ++l;
    return l;
}

// Row path layout of a fused item's destinations: sub-group g of `split` owns
// slots g * (DL_FAN / split) onwards and gets destinations g * per ..
// g * per + per - 1 (per = ceil(k / split)), filled from the front; unused
// slots are null, which is what ends a sub-group's store loop on the device.
inline void slots_by_subgroup(dl_plain_item &, uint32_t) {}
inline void slots_by_subgroup(dl_fused_item &it, uint32_t split)
{
    char *by_group[DL_FAN] = {};
    const uint32_t slots = (uint32_t)DL_FAN / split, per = (it.k + split - 1) / split;
    for (uint32_t g = 0; g < split; ++g)
        for (uint32_t q = 0; q < per && g * per + q < it.k; ++q) by_group[g * slots + q] = it.dst[g * per + q];
    for (int j = 0; j < DL_FAN; ++j) it.dst[j] = by_group[j];
}

inline uint32_t item_k(const dl_plain_item &) { return 1; }
inline uint32_t item_k(const dl_fused_item &it) { return it.k; }

constexpr uint32_t ARMED_DIRECT_MAX = 16;  // grids up to this size report in a completion word per workgroup; the shape rule below aims for them

// Workgroups of an armed kernel.  While it waits for its doorbell the kernel must leave room for other
// kernels, above all for the ones that produce what it is going to copy.  Room means whole compute units: a
// kernel whose wavefronts take all the vector registers of a SIMD (a large matrix multiplication's do) cannot
// share that SIMD with even one waiting wavefront, and behind a grid that had a workgroup on every compute
// unit such a kernel did not start until the armed request expired.  Unless the caller sets the cap, the grid
// has at most one workgroup for every other compute unit.
// A kernel that does not wait (signal mode) is in nobody's way: it gets half of the wavefront slots.
uint32_t armed_grid(uint64_t tiles, uint32_t block_threads, bool waits)
{
    const uint32_t cus = (uint32_t)(g_dl.num_cu > 0 ? g_dl.num_cu : 256);
    uint32_t cap = g_dl.cfg.armed_blocks ? g_dl.cfg.armed_blocks : waits ? cus / 2u : 16u * cus / (block_threads / 64u);
    if (cap < 1u) cap = 1u;
    if (cap > 32768u) cap = 32768u;  // the arrival counter keeps 16 bits for the count
    return (uint32_t)(tiles < cap ? tiles : cap);
}

// Enqueue the gate of a chained request and turn `a` into what the copy kernel behind it gets.
int launch_gate(dl_arm &a, hipStream_t stream)
{
    dl_arm gate = a;
    gate.direct = 1;  // one workgroup: it polls the doorbell itself wherever that lies
    gate.own_word = 0;
    gate.gated = 0;
    hipLaunchKernelGGL(dl_arm_gate_kernel, dim3(1), dim3(64), 0, stream, gate);
    DL_HIP(hipGetLastError());
    a.nowait = 1;
    a.gated = 1;
    return DL_OK;
}

template <class Item, int NMAX>
int launch_klist(const Item *items, size_t n, const uint64_t *tile_end, const dl_launch_shape &sh, hipStream_t stream,
                 const dl_arm *arm)
{
    dl_klist<Item, NMAX> p;
    p.n = (uint32_t)n;
    p.tile_bytes = sh.tile_bytes;
    p.split = sh.split;
    p.split_log2 = log2u(sh.split);
    p.wpg_log2 = log2u(sh.block_threads / 64u / sh.split);
    for (size_t i = 0; i < n; ++i) {
        p.tile_end[i] = (uint32_t)tile_end[i];
        p.item[i] = items[i];
    }
    for (size_t i = n; i < (size_t)NMAX; ++i) p.tile_end[i] = 0xFFFFFFFFu;  // the device compares without looking at n
    const bool on_grid = all_on_grid(items, n);
    if constexpr (std::is_same<Item, dl_fused_item>::value) {
        if (sh.pairs) {  // (tile_end counts workgroups: one per row and pair of destinations)
            const uint32_t blocks = (uint32_t)tile_end[n - 1];
            dl_with_policy_and_grid(sh.policy, on_grid, [&](auto pol, auto og) {
                hipLaunchKernelGGL((dl_exec_pairs_kernel<NMAX, decltype(pol)::value, decltype(og)::value>), dim3(blocks),
                                   dim3(64), 0, stream, p);
            });
            DL_HIP(hipGetLastError());
            return DL_OK;
        }
    }
    if (sh.rows)
        for (size_t i = 0; i < n; ++i) slots_by_subgroup(p.item[i], sh.split);
    const uint32_t grid = (uint32_t)tile_end[n - 1];
    if (arm) {
        dl_arm a = *arm;
        if (sh.chain && !a.nowait) {
            const int rc = launch_gate(a, stream);
            if (rc != DL_OK) return rc;
        }
        const bool signal = sh.rows && a.nowait && !a.gated && !g_dl.cfg.armed_blocks && grid <= SIGNAL_MAX_BLOCKS;
        const uint32_t g = signal ? grid : armed_grid(grid, sh.block_threads, !a.nowait);
        a.direct = g <= a.direct_max ? 1u : 0u;
        a.own_word = g <= DL_DONE_WORDS && !a.trace_host ? 1u : 0u;  // the stamps come from the last arriver
        g_dl.armed_words = a.own_word ? g : 1u;
        g_dl.armed_counted = !a.own_word;
        if (signal && on_grid)
            hipLaunchKernelGGL((dl_signal_rows_kernel<Item, NMAX, true>), dim3(g), dim3(sh.block_threads), 0, stream, p, a);
        else if (signal)
            hipLaunchKernelGGL((dl_signal_rows_kernel<Item, NMAX, false>), dim3(g), dim3(sh.block_threads), 0, stream, p, a);
        else if (sh.rows && !a.nowait && a.direct && sh.split == 1 && (grid <= 4u * g || sh.block_threads > 512u) && !std::is_same<Item, dl_swap_item>::value) {
            if constexpr (!std::is_same<Item, dl_swap_item>::value) {
                const bool four = grid > (sh.block_threads > 512u ? 4u : 2u) * g;  // (see dl_armed_passes_kernel)
                const auto kernel = g < grid ? four ? dl_armed_passes_kernel<Item, NMAX, 4> : dl_armed_passes_kernel<Item, NMAX, 2>
                                    : on_grid ? dl_armed_rows_kernel<Item, NMAX, true> : dl_armed_rows_kernel<Item, NMAX, false>;
                hipLaunchKernelGGL(kernel, dim3(g), dim3(sh.block_threads), 0, stream, p, a);
            }
        } else if (sh.block_threads > 512u)
            return DL_ERR_INVALID;  // not for the kernels below (and no shape rule asks for it)
        else if (sh.rows)
            hipLaunchKernelGGL((dl_armed_list_kernel<Item, NMAX, true>), dim3(g), dim3(sh.block_threads), 0, stream, p, a);
        else
            hipLaunchKernelGGL((dl_armed_list_kernel<Item, NMAX, false>), dim3(g), dim3(sh.block_threads), 0, stream, p, a);
    } else if (sh.rows && sh.rows2d_width && sh.eighths) {
        if constexpr (std::is_same<Item, dl_plain_item>::value)
            hipLaunchKernelGGL((dl_exec_rows2d_kernel<Item, NMAX, DL_POL_WT, false, true>), dim3((uint32_t)dl_eighths_width(sh.rows2d_width), (uint32_t)n),
                               dim3(sh.block_threads), 0, stream, p);
    } else if (sh.rows && sh.rows2d_width) {
        dl_with_policy_and_grid(sh.policy, on_grid, [&](auto pol, auto og) {
            hipLaunchKernelGGL((dl_exec_rows2d_kernel<Item, NMAX, decltype(pol)::value, decltype(og)::value>),
                               dim3(sh.rows2d_width, (uint32_t)n), dim3(sh.block_threads), 0, stream, p);
        });
    } else if (sh.rows) {
        dl_with_policy_and_grid(sh.policy, on_grid, [&](auto pol, auto og) {
            hipLaunchKernelGGL((dl_exec_rows_kernel<Item, NMAX, decltype(pol)::value, decltype(og)::value>), dim3(grid),
                               dim3(sh.block_threads), 0, stream, p);
        });
    } else if (sh.max_blocks && grid > sh.max_blocks) {
        dl_with_policy(sh.policy, [&](auto pol) {
            hipLaunchKernelGGL((dl_exec_list_strided_kernel<Item, NMAX, decltype(pol)::value>), dim3(sh.max_blocks),
                               dim3(sh.block_threads), 0, stream, p);
        });
    } else {
        dl_with_policy(sh.policy, [&](auto pol) {
            hipLaunchKernelGGL((dl_exec_list_kernel<Item, NMAX, decltype(pol)::value>), dim3(grid),
                               dim3(sh.block_threads), 0, stream, p);
        });
    }
    DL_HIP(hipGetLastError());
    return DL_OK;
}

inline void advance(dl_plain_item &it, uint64_t off)
{
    it.src += off;
    it.dst += off;
}
inline void advance(dl_fused_item &it, uint64_t off)
{
    it.src += off;
    for (uint32_t j = 0; j < it.k; ++j) it.dst[j] += off;
}

// Short tables skip the pinned ring.  Where the device exposes all of its memory through a PCIe BAR the host
// writes the table straight into device memory (write-combined stores, nothing is ever read back), fences, and
// launches: posted writes reach the device in order, the launch's doorbell is one of them, so the kernel finds
// the table complete, and in its own memory.  (Through the pinned ring every workgroup fetched its entry over
// the host link, or a staging kernel ran in front.)
//
// push_acquire: a slot for a table of table_bytes whose kernel will be launched on `stream` next, or null if
// this table cannot go that way (*rc says whether that is an error).  push_commit: after that launch.
// Wait for `ev`, behind which the memory that is about to be reused was last read.  If that reader is an armed
// request that nobody has triggered yet, the wait could only end with that request's expiry: refuse instead.
int wait_for_readers(hipEvent_t ev, uint64_t armed_ticket)
{
    if (armed_ticket && dl_armed_untriggered(armed_ticket)) return DL_ERR_STATE;
    DL_HIP(hipEventSynchronize(ev));
    return DL_OK;
}

// Record one event behind everything the open batch has launched; its slots are covered by it from now on.
int push_close_batch()
{
    if (g_ring.batch_len == 0) return DL_OK;
    const size_t last = (g_ring.batch_first + g_ring.batch_len - 1) % PUSH_SLOTS;
    DL_HIP(hipEventRecord(g_ring.push_ev[last], g_ring.batch_stream));
    for (size_t q = 0; q < g_ring.batch_len; ++q) g_ring.push_cover[(g_ring.batch_first + q) % PUSH_SLOTS] = (int)last;
    g_ring.batch_len = 0;
    return DL_OK;
}

char *push_acquire(size_t table_bytes, hipStream_t stream, int *rc)
{
    *rc = DL_OK;
    if (!g_ring.push || !g_dl.cfg.table_push || table_bytes > PUSH_PAYLOAD_BYTES) return nullptr;
    // a batch is one stream's: another stream ends it (on its own stream, which is one that cannot have gone)
    if (g_ring.batch_len && (stream != g_ring.batch_stream || g_ring.batch_len >= PUSH_BATCH))
        if ((*rc = push_close_batch()) != DL_OK) return nullptr;
    const size_t s = g_ring.push_next;
    if (g_ring.push_used[s]) {  // the kernel that read this slot's previous table must have ended
        if (g_ring.push_cover[s] < 0) {
            *rc = DL_ERR_STATE;  // cannot happen: a batch is shorter than the ring
            return nullptr;
        }
        if ((*rc = wait_for_readers(g_ring.push_ev[g_ring.push_cover[s]], g_ring.push_armed[s])) != DL_OK) return nullptr;
    }
    g_ring.push_used[s] = false;  // free until push_commit: a call that fails in between leaves it so
    g_ring.push_armed[s] = 0;
    return g_ring.push + s * PUSH_SLOT_BYTES;
}

// After the last write into the slot: the payload leaves the write-combining buffers, then the stamp, then
// whatever the caller does next (the launch).
uint64_t push_seal(char *slot)
{
    static uint64_t stamps = 0;
    const uint64_t stamp = ++stamps;
    _mm_sfence();
    *(volatile uint64_t *)(slot + PUSH_PAYLOAD_BYTES) = stamp;
    _mm_sfence();
    return stamp;
}

// After the launch that reads the slot push_acquire gave out last (only then is the slot taken).  armed_ticket: that launch is a request armed
// in prelaunch mode (0: it is not).
int push_commit(hipStream_t stream, uint64_t armed_ticket)
{
    const size_t s = g_ring.push_next;
    g_ring.push_next = (s + 1) % PUSH_SLOTS;
    g_ring.push_used[s] = true;
    g_ring.push_cover[s] = -1;
    g_ring.push_armed[s] = armed_ticket;
    if (stream == nullptr || stream == g_ring.own_stream) {
        if (g_ring.batch_len == 0) {
            g_ring.batch_first = s;
            g_ring.batch_stream = stream;
        }
        ++g_ring.batch_len;
        return DL_OK;
    }
    // a caller's stream: it may be gone by the next call, so its event is recorded now
    DL_HIP(hipEventRecord(g_ring.push_ev[s], stream));
    g_ring.push_cover[s] = (int)s;
    return DL_OK;
}

// Copy `bytes` (a multiple of 16) from a slot of the pinned ring to the same slot of its device
// mirror with a 1:1 row kernel of our own, enqueued on `stream` in front of the kernel that reads it.
int stage_slot(size_t s, uint64_t bytes, hipStream_t stream)
{
    dl_plain_item stage{g_ring.base + s * RING_SLOT_BYTES, g_ring.dev + s * RING_SLOT_BYTES, bytes};
    dl_launch_shape ssh = dl_choose_shape(stage.bytes, stage.bytes, 1);
    ssh.split = 1;
    ssh.tile_bytes = 16u * ssh.block_threads;  // the row path's tile: one 1 KiB row per wavefront
    ssh.rows = true;
    uint64_t stage_tiles = dl_item_tiles(stage, ssh.tile_bytes);
    return launch_klist<dl_plain_item, NMAX_SMALL>(&stage, 1, &stage_tiles, ssh, stream, nullptr);
}

// The cache policy of a list of plain copies or swaps that choose_shape gave streaming loads, once it is known how it is
// executed (rows: by the row path with the list in the kernel arguments).
//  - Where a source and its destination differ modulo 16 (aligned: no item's do), the loads of neighbouring lanes and
//    rows meet inside 16-byte words, and a streaming load leaves nothing of them in a cache: it pays only where the rows of
//    an item are in flight together.  Lists of unequal copies, 181 / 755 MiB moved, one buffer set / three in turn,
//    write-through stores alone against streaming loads: 24.8 / 34.3 and 135 / 134 us against 32.6 / 34.5 and
//    143 / 143; 100 of them (a table), 201 MiB 27.4 / 45.4 against 39.1 / 47.0; 1000 equal ones of 60 KiB 20.1 / 27.3
//    against 27.9 / 27.9; swaps, 224 and 896 MiB 30.1 / 40.1 and 153 / 155 against 37.2 / 43.6 and 160 / 161.
//  - Else, lists that do not take the row path do best with the hint on both sides from 512 MiB moved: all-to-all of
//    unequal chunks, 518 / 1036 MiB moved 88.3 / 174 us against 92.5 / 182; 8000 equal copies of 60 KiB 172 : 182, a
//    table of 300 unequal ones, 584 MiB 124 : 128 (with one buffer set 123 : 119).
template <class Item>
int plain_policy(int policy, bool rows, bool aligned, uint64_t moved)
{
    if (policy != DL_POL_STREAM_IN) return policy;
    if (!aligned) return rows && !std::is_same<Item, dl_swap_item>::value ? DL_POL_STREAM_IN : DL_POL_WT;
    return !rows && moved >= STREAM_BOTH_MIN_BYTES ? DL_POL_STREAM : DL_POL_STREAM_IN;
}

template <class Item>
bool all_aligned(const Item *items, size_t n)
{
    for (size_t i = 0; i < n; ++i)
        if (((uint64_t)items[i].src ^ (uint64_t)items[i].dst) & 15u) return false;
    return true;
}

// Equally long plain copies or swaps that do not fit a dl_klist but whose offsets do fit the kernel arguments (up to
// 480): one launch and nothing else.  Returns false if the list does not qualify (and nothing was enqueued).
template <class Item, int NMAX>
int launch_offsets_sized(const Item *items, size_t n, const dl_offset_head &head, uint32_t width, uint32_t threads, int policy,
                         bool on_grid, bool eighths, hipStream_t stream)
{
    dl_offset_list<NMAX> p;
    static_cast<dl_offset_head &>(p) = head;
    for (size_t i = 0; i < n; ++i) {
        p.at[i].src = (uint32_t)((uint64_t)(items[i].src - head.src) >> head.unit_log2);
        p.at[i].dst = (uint32_t)((uint64_t)(items[i].dst - head.dst) >> head.unit_log2);
    }
    if (eighths) {
        if constexpr (std::is_same<Item, dl_plain_item>::value)
            hipLaunchKernelGGL((dl_exec_offsets_kernel<Item, NMAX, DL_POL_WT, false, true>), dim3((uint32_t)dl_eighths_width(width), (uint32_t)n),
                               dim3(threads), 0, stream, p);
    } else
        dl_with_policy_and_grid(policy, on_grid, [&](auto pol, auto og) {
            hipLaunchKernelGGL((dl_exec_offsets_kernel<Item, NMAX, decltype(pol)::value, decltype(og)::value>), dim3(width, (uint32_t)n),
                               dim3(threads), 0, stream, p);
        });
    DL_HIP(hipGetLastError());
    return DL_OK;
}

template <class Item>
bool launch_offsets(const Item *items, size_t n, const dl_launch_shape &sh, hipStream_t stream, int *rc)
{
    const dl_config &c = g_dl.cfg;
    constexpr int SMALL = 256, BIG = 480;
    static_assert(sizeof(dl_offset_list<BIG>) <= 4096, "kernel arguments");
    if (c.tile_bytes || c.block_threads || sh.max_blocks) return false;
    // A longer list takes several launches if each of them has enough to do to hide the kernel start in between
    // (512 blocks of 512 KiB: 98.5 us from a table, 87.6 in two launches).
    const size_t launches = (n + BIG - 1) / BIG, per = (n + launches - 1) / launches;
    if (launches > 1 && 2u * items[0].bytes * per < OFFSETS_MIN_BYTES) return false;
    // the addresses relative to the lowest one of each side: 16-byte units if all of them agree modulo 16, else bytes
    const char *src = items[0].src, *src_hi = src, *dst = items[0].dst, *dst_hi = dst;
    uint64_t apart = 0, any_src = 0, any_dst = 0, across = 0;
    uint32_t worst = 0;  // how far behind its grid the worst first destination lies
    const uint64_t bytes = items[0].bytes;
    for (size_t i = 0; i < n; ++i) {
        const Item &it = items[i];
        if (it.bytes != bytes) return false;
        src = it.src < src ? it.src : src;
        src_hi = it.src > src_hi ? it.src : src_hi;
        dst = it.dst < dst ? it.dst : dst;
        dst_hi = it.dst > dst_hi ? it.dst : dst_hi;
        any_src |= (uint64_t)it.src;
        any_dst |= (uint64_t)it.dst;
        across |= (uint64_t)it.src ^ (uint64_t)it.dst;
        apart |= ((uint64_t)it.src ^ (uint64_t)items[0].src) | ((uint64_t)it.dst ^ (uint64_t)items[0].dst);
        const uint32_t shift = dl_item_shift(it);
        worst = shift > worst ? shift : worst;
    }
    const bool on_grid = (any_dst & (DL_CUT - 1u)) == 0 && (any_src & 3u) == 0 && (bytes & 15u) == 0;  // (item_on_grid for all)
    dl_offset_head head;
    head.unit_log2 = (apart & 15u) ? 0u : 4u;
    if (((uint64_t)(src_hi - src) >> head.unit_log2) >> 32 || ((uint64_t)(dst_hi - dst) >> head.unit_log2) >> 32) return false;
    const uint32_t threads = sh.block_threads, tile = 16u * threads;
    const uint64_t width = (bytes + worst + tile - 1u) / tile;  // of that item; the others may leave a workgroup without work
    if (width * n >= (1ull << 30) || width * threads >= (1ull << 32)) return false;
    head.src = src;
    head.dst = (char *)dst;
    head.bytes = bytes;
    head.wpg_log2 = log2u(threads / 64u);
    const int policy = plain_policy<Item>(sh.policy, true, (across & 15u) == 0, 2u * bytes * n);
    *rc = DL_OK;
    for (size_t i = 0; i < n && *rc == DL_OK; i += per) {
        const size_t m = n - i < per ? n - i : per;
        *rc = m <= (size_t)SMALL
                  ? launch_offsets_sized<Item, SMALL>(items + i, m, head, (uint32_t)width, threads, policy, on_grid, sh.eighths, stream)
                  : launch_offsets_sized<Item, BIG>(items + i, m, head, (uint32_t)width, threads, policy, on_grid, sh.eighths, stream);
    }
    return true;
}

// Long list of equally sized items that moves enough bytes to pay for staging
// its table: the items themselves (not cut into tiles) go to device memory and the row kernel
// above works on them.  Returns false if the list does not qualify.  (Lists that fit the kernel arguments,
// such as the 64 chunks of a uniform all-to-all, and equal plain copies at offsets that do, see launch_offsets,
// never come here: from there they need no table.)
template <class Item>
bool launch_uniform_rows(const Item *items, size_t n, const dl_launch_shape &sh, hipStream_t stream, int *rc)
{
    const dl_config &c = g_dl.cfg;
    if (c.tile_bytes || sh.max_blocks) return false;
    // Read-once/write-k items with a mix of fan-outs (token rows: 1 to 8 destinations, 5.3 on average) go
    // fastest with two wavefronts per 1 KiB row, each storing to up to four destinations, in workgroups of
    // just those two: 5-20 % faster over mean fan-outs 1.9 .. 8 than four wavefronts with two stores each,
    // of which the ones without a destination are dead weight at the rate wavefronts can be started.
    const bool fused = std::is_same<Item, dl_fused_item>::value;
    const uint32_t split = c.fan_split ? sh.split : fused ? DL_TABLE_ROWS_SPLIT : 1u;
    if (n * sizeof(Item) > RING_SLOT_BYTES) return false;
    const uint64_t bytes = items[0].bytes;
    uint32_t kmax = 1, worst = 0;  // how far behind its grid the worst first destination lies
    uint64_t any_src = 0, across = 0;
    for (size_t i = 0; i < n; ++i) {
        if (items[i].bytes != bytes) return false;
        if (item_k(items[i]) > kmax) kmax = item_k(items[i]);
        const uint32_t shift = dl_item_shift(items[i]);
        worst = shift > worst ? shift : worst;
        any_src |= (uint64_t)items[i].src;
        if constexpr (!std::is_same<Item, dl_fused_item>::value) across |= (uint64_t)items[i].src ^ (uint64_t)items[i].dst;
    }
    const bool on_grid = worst == 0 && (any_src & 3u) == 0 && (bytes & 15u) == 0;  // (item_on_grid for all)
    const bool aligned = (across & 15u) == 0;
    // a table that needs staging must move enough bytes to pay for it; one written through the BAR needs none.
    // But every workgroup that reads a pushed table looks for the stamp and fetches its entry past the caches, two
    // round trips that cost a large request 12 % of its kernel time, against 4 us for the staging kernel and the
    // gap behind it: from UNIFORM_ROWS_STAGE_BYTES moved, the table is staged (256 copies of 4 MiB: 368 -> 345 us).
    const bool pushable = g_ring.push && c.table_push && n * sizeof(Item) <= PUSH_PAYLOAD_BYTES &&
                          bytes * n * (1u + kmax) < UNIFORM_ROWS_STAGE_BYTES;
    if (!pushable && bytes * n < UNIFORM_ROWS_MIN_BYTES) return false;
    // Plain items: one wavefront per workgroup as in shorter lists of that size, but not where every workgroup first
    // fetches its entry of a pushed table, unless the loads are unaligned.  Four wavefronts against one, three buffer
    // sets in turn: staged, 3000 / 8000 / 20 000 copies of 60 KiB 72.5 / 176 / 436 us against 72.1 / 173 / 427,
    // unaligned 77.1 / 194 and 72.6 / 184; pushed, 1000 copies 22.2 against 23.3, unaligned 30.6 against 27.3.
    const bool waves = !fused && (!pushable || !aligned) && dl_plain_threads(2u * bytes * n, false) == 64u;
    const uint32_t threads = c.block_threads ? c.block_threads : fused && !c.fan_split ? DL_TABLE_ROWS_THREADS : waves ? 64u : 256u;
    if (threads > 512u || threads % (64u * split) || ((threads / 64u / split) & (threads / 64u / split - 1u)))
        return false;  // whole sub-groups of a power-of-two number of wavefronts
    const int policy = fused ? sh.policy : plain_policy<Item>(sh.policy, false, aligned, 2u * bytes * n);
    const uint32_t tile = 16u * threads / split;  // one 1 KiB row per wavefront of a sub-group
    const uint64_t tpi = (bytes + worst + tile - 1u) / tile;  // of the item that lies worst on its grid; the others leave a workgroup without work
    if (tpi * n >= (1ull << 30) || tpi >= (1ull << 31) || n > DL_UROWS_MAX_ITEMS) return false;

    char *pushed = pushable ? push_acquire(n * sizeof(Item), stream, rc) : nullptr;
    if (*rc != DL_OK) return true;
    size_t s = 0;
    *rc = DL_ERR_HIP;
    if (!pushed) {
        s = g_ring.next++ % RING_SLOTS;
        if (g_ring.used[s]) {
            if ((*rc = wait_for_readers(g_ring.ev[s], g_ring.armed[s])) != DL_OK) {
                --g_ring.next;
                return true;
            }
            *rc = DL_ERR_HIP;
        }
        g_ring.armed[s] = 0;
    }
    Item *slot = (Item *)(pushed ? pushed : g_ring.base + s * RING_SLOT_BYTES);
    for (size_t i = 0; i < n; ++i) {
        Item it = items[i];
        slots_by_subgroup(it, split);
        slot[i] = it;  // write only: the slot may be device memory behind the BAR
    }
    const Item *dslot = slot;
    uint64_t stamp = 0;
    if (pushed) {
        stamp = push_seal(pushed);
    } else {
        *rc = stage_slot(s, (n * sizeof(Item) + 15u) & ~(uint64_t)15u, stream);
        if (*rc != DL_OK) return true;
        dslot = (const Item *)(g_ring.dev + s * RING_SLOT_BYTES);
    }
    const dl_pushed ps = dl_push_kernel_args(stamp);
    dl_with_policy_and_grid(policy, on_grid, [&](auto pol, auto og) {
        if (pushed)
            hipLaunchKernelGGL((dl_exec_urows_kernel<Item, decltype(pol)::value, true, decltype(og)::value>),
                               dim3((uint32_t)tpi, (uint32_t)n), dim3(threads), 0, stream, dslot,
                               log2u(threads / 64u / split), log2u(split), ps);
        else
            hipLaunchKernelGGL((dl_exec_urows_kernel<Item, decltype(pol)::value, false, decltype(og)::value>),
                               dim3((uint32_t)tpi, (uint32_t)n), dim3(threads), 0, stream, dslot,
                               log2u(threads / 64u / split), log2u(split), ps);
    });
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !pushed) e = hipEventRecord(g_ring.ev[s], stream);
    if (e != hipSuccess) {
        g_dl.last_hip = (int)e;
        *rc = DL_ERR_HIP;
        return true;
    }
    if (pushed) {
        *rc = push_commit(stream, 0);
        return true;
    }
    g_ring.used[s] = true;
    *rc = DL_OK;
    return true;
}

template <class Item>
int launch_table(const Item *items, size_t n, dl_launch_shape sh, hipStream_t stream, const dl_arm *arm)
{
    if (!g_ring.base) return DL_ERR_STATE;
    if (!arm) {
        int rc = DL_OK;
        if (launch_uniform_rows(items, n, sh, stream, &rc)) return rc;
    }
    if constexpr (!std::is_same<Item, dl_fused_item>::value) {
        if (sh.policy == DL_POL_STREAM_IN) {
            uint64_t moved = 0;
            for (size_t i = 0; i < n; ++i) moved += 2u * items[i].bytes;
            sh.policy = plain_policy<Item>(sh.policy, false, all_aligned(items, n), moved);
        }
    }
    const size_t cap = RING_SLOT_BYTES / sizeof(Item);
    auto entries = [&](uint32_t tile) {  // one per tile of the first destination's grid, like everywhere
        uint64_t m = 0;
        for (size_t i = 0; i < n; ++i) m += dl_item_tiles(items[i], tile);
        return m;
    };
    // Entries are what a long list pays for (a table in the pinned ring: every workgroup fetches its
    // entry over the host link, ~1.5 us each, a few hundred in flight): with one entry per 4 KiB,
    // 256 copies of 1 MiB ran at 2.3 TB/s and 256 copies of 16 KiB took 11.6 us.  Unless the caller
    // fixed the tile: one entry per item up to 64 KiB (7.6 us for the same 256 copies), 64 KiB tiles
    // for larger items (4.7 TB/s), and coarser still when that leaves more than a few thousand
    // entries.  The workgroup loops over its tile.  (With the table in device memory, through the BAR,
    // tiles from 4 to 64 KiB were within 1 us of each other; the same rule is kept.)
    if (g_dl.cfg.tile_bytes == 0) {
        uint64_t biggest = 0;
        for (size_t i = 0; i < n; ++i) biggest = items[i].bytes > biggest ? items[i].bytes : biggest;
        while (sh.tile_bytes < 65536u && sh.tile_bytes < biggest) sh.tile_bytes *= 2;
        sh.block_threads = 256;
        if (sh.block_threads / sh.split < 64) sh.split = 1;
    }
    while (sh.tile_bytes < (1u << 20) && entries(sh.tile_bytes) > TABLE_ENTRIES_TARGET) sh.tile_bytes *= 2;
    if (arm) {
        // an armed request is exactly one kernel: grow the tile until the cut list fits one ring slot
        while (entries(sh.tile_bytes) > cap) {
            if (sh.tile_bytes >= (1u << 30)) return DL_ERR_INVALID;
            sh.tile_bytes *= 2;
        }
    }
    const uint64_t all_entries = entries(sh.tile_bytes);
    size_t i = 0;
    uint64_t off = 0;  // progress inside items[i]
    while (i < n) {
        // a short table that is all of the request
        char *pushed = nullptr;
        uint64_t pushed_armed_ticket = 0;
        if (i == 0 && off == 0) {
            int rc = DL_OK;
            pushed = push_acquire(all_entries * sizeof(Item), stream, &rc);
            if (rc != DL_OK) return rc;
        }
        size_t s = 0;
        if (!pushed) {
            s = g_ring.next++ % RING_SLOTS;
            if (g_ring.used[s]) {
                const int rc = wait_for_readers(g_ring.ev[s], g_ring.armed[s]);
                if (rc != DL_OK) {
                    --g_ring.next;
                    return rc;
                }
            }
            g_ring.armed[s] = 0;
        }
        Item *slot = (Item *)(pushed ? pushed : g_ring.base + s * RING_SLOT_BYTES);
        size_t m = 0;
        while (i < n && m < cap) {
            const uint64_t left = items[i].bytes - off;
            if (left == 0) {
                ++i;
                off = 0;
                continue;
            }
            Item it = items[i];
            advance(it, off);
            const uint64_t room = sh.tile_bytes - dl_item_shift(it);  // up to the next tile boundary of the grid
            it.bytes = left < room ? left : room;
            slot[m++] = it;  // write only: the slot may be device memory behind the BAR
            off += it.bytes;
        }
        if (m == 0) break;
        uint64_t stamp = 0;
        if (pushed) {
            stamp = push_seal(pushed);
        } else if (m >= TABLE_STAGE_MIN) {
            // Stage the table in device memory, in front of the kernel that uses it (the copy does not
            // wait for a doorbell: the table is final now).  The workgroups then find their entries in
            // HBM instead of each fetching one over the host link.
            const int rc = stage_slot(s, (m * sizeof(Item) + 15u) & ~(uint64_t)15u, stream);
            if (rc != DL_OK) return rc;
            slot = (Item *)(g_ring.dev + s * RING_SLOT_BYTES);
        }
        const dl_pushed ps = dl_push_kernel_args(stamp);
        if (arm) {
            dl_arm a = *arm;
            if (sh.chain && !a.nowait) {
                const int rc = launch_gate(a, stream);
                if (rc != DL_OK) return rc;
            }
            const uint32_t g = armed_grid(m, sh.block_threads, !a.nowait);
            a.direct = g <= a.direct_max ? 1u : 0u;
            a.own_word = g <= DL_DONE_WORDS && !a.trace_host ? 1u : 0u;
            g_dl.armed_words = a.own_word ? g : 1u;
            g_dl.armed_counted = !a.own_word;
            if (pushed)
                hipLaunchKernelGGL((dl_armed_table_kernel<Item, true>), dim3(g), dim3(sh.block_threads), 0, stream, slot,
                                   (uint32_t)m, sh.split, ps, a);
            else
                hipLaunchKernelGGL((dl_armed_table_kernel<Item, false>), dim3(g), dim3(sh.block_threads), 0, stream, slot,
                                   (uint32_t)m, sh.split, ps, a);
            // whoever wants this memory next must not wait for a request that nobody has triggered
            // (arm->nowait: a chained request's copy kernel does not wait itself, but its gate does)
            if (!arm->nowait) {
                if (pushed)
                    pushed_armed_ticket = a.ticket;
                else
                    g_ring.armed[s] = a.ticket;
            }
        } else {
            dl_with_policy(sh.policy, [&](auto pol) {
                if (pushed)
                    hipLaunchKernelGGL((dl_exec_table_kernel<Item, decltype(pol)::value, true>), dim3((uint32_t)m),
                                       dim3(sh.block_threads), 0, stream, slot, (uint32_t)m, sh.split, ps);
                else
                    hipLaunchKernelGGL((dl_exec_table_kernel<Item, decltype(pol)::value, false>), dim3((uint32_t)m),
                                       dim3(sh.block_threads), 0, stream, slot, (uint32_t)m, sh.split, ps);
            });
        }
        DL_HIP(hipGetLastError());
        if (pushed) {
            const int rc = push_commit(stream, pushed_armed_ticket);
            if (rc != DL_OK) return rc;
            continue;
        }
        DL_HIP(hipEventRecord(g_ring.ev[s], stream));
        g_ring.used[s] = true;
    }
    return DL_OK;
}

template <class Item>
int exec_list(const Item *items, size_t n, hipStream_t stream, const dl_arm *arm, bool *launched)
{
    *launched = false;
    if (n == 0) return DL_OK;
    uint64_t total = 0, biggest = 0;
    uint32_t kmax = 1;
    for (size_t i = 0; i < n; ++i) {
        total += items[i].bytes;
        if (items[i].bytes > biggest) biggest = items[i].bytes;
        if (item_k(items[i]) > kmax) kmax = item_k(items[i]);
    }
    if (total == 0) return DL_OK;
    dl_launch_shape sh = dl_choose_shape(total, biggest, kmax);
    // A signalled request that moves more than a little is an ordinary one-shot request, and a kernel of one workgroup behind
    // it reports: the copy then has a full grid, loads that the caches may serve and no count at its end, for the second
    // launch's 2 us.  Issue to done and the call, one kernel : two, all-gather over eight ranks 128 / 256 KiB per rank 11.6 / 12.5 :
    // 11.6 / 12.3 us, 1 / 2 MiB 19.4 / 39.4 : 19.2 / 36.2, over sixteen 1 / 2 MiB 66 / 122 : 55 / 100; all-to-all over eight of
    // 64 KiB chunks (8 MiB moved) 12.0 : 12.4, 128 / 256 KiB 13.0 / 16.9 : 12.4 / 15.2, 1 MiB 37.1 : 30.0.  (Not with stores that
    // stay in the L2, nor where the caller has fixed the armed grid or wants the phase stamps.)
    if (arm && arm->nowait && !arm->trace_host && !g_dl.cfg.armed_blocks && sh.policy != DL_POL_PLAIN && !sh.max_blocks) {
        uint64_t moved = 0;
        for (size_t i = 0; i < n; ++i)
            moved += items[i].bytes * (std::is_same<Item, dl_swap_item>::value ? 4ull : 1ull + item_k(items[i]));
        if (moved >= SIGNAL_DONE_MIN_BYTES) {
            // (not what needs a table: a kernel that gave up on its table would be reported as done)
            int rc = DL_OK;
            bool sent = false;
            if (n <= (size_t)list_cap<Item>::big)
                rc = exec_list(items, n, stream, nullptr, &sent);
            else if constexpr (!std::is_same<Item, dl_fused_item>::value)
                sent = launch_offsets(items, n, sh, stream, &rc);
            if (rc != DL_OK) return rc;
            if (sent) {
                hipLaunchKernelGGL(dl_signal_done_kernel, dim3(1), dim3(64), 0, stream, arm->done, arm->ticket);
                DL_HIP(hipGetLastError());
                g_dl.armed_words = 1;
                g_dl.armed_counted = false;
                *launched = true;
                return DL_OK;
            }
        }
    }
    // one-shot requests, where the caller has not fixed the shape
    const bool free_shape = !arm && !g_dl.cfg.tile_bytes && !g_dl.cfg.block_threads && !g_dl.cfg.fan_split && !sh.max_blocks;
    if (arm && !arm->nowait && g_dl.cfg.armed_blocks == 0) {
        // prelaunch mode, and the caller has not fixed the waiting grid: large requests wait in a gate kernel
        uint64_t moved = 0;
        for (size_t i = 0; i < n; ++i)
            moved += items[i].bytes * (std::is_same<Item, dl_swap_item>::value ? 4ull : 1ull + item_k(items[i]));
        sh.chain = moved > g_dl.cfg.armed_chain_min_bytes;
    }
    if (arm && g_dl.cfg.tile_bytes == 0 && g_dl.cfg.block_threads == 0) {
        // armed kernels pay per workgroup for the doorbell fan-out and the arrival count:
        // four wavefronts per workgroup, each still moving 1 KiB rows
        sh.tile_bytes = 4096;
        sh.block_threads = biggest >= 4096 ? 256u : sh.block_threads;
        sh.split = 1;
        // Up to ARMED_DIRECT_MAX workgroups report each in a completion word of its own, and with the doorbell
        // in host memory only that many poll it themselves (32 or 64 pollers over the link took 7 and 9.5 us,
        // the hop through device flags 6.5, against 5.0-5.2).  A request too long for that takes eight
        // wavefronts per workgroup where that cuts the number of workgroups: more of them stay below the limit,
        // and above it arrivals and passes over a capped grid halve (1 MiB per rank: 17.1 -> 14.6 us).
        uint64_t t4 = 0, t8 = 0;
        for (size_t i = 0; i < n; ++i) {
            t4 += dl_item_tiles(items[i], 4096);
            t8 += dl_item_tiles(items[i], 8192);
        }
        if (sh.block_threads == 256u && t4 > ARMED_DIRECT_MAX && 3u * t8 <= 2u * t4) {
            sh.tile_bytes = 8192;
            sh.block_threads = 512;
        }
        // A waiting grid is capped in workgroups, so where eight wavefronts each would make several passes it takes sixteen:
        // only in the kernels whose workgroups all poll the doorbell themselves, the others being built for 512 threads.
        // All-gather over eight ranks, trigger to done and the call, 256 KiB / 1 MiB per rank 16.6 / 25.3 us with eight,
        // 15.4 / 24.6 with sixteen.
        if (!std::is_same<Item, dl_swap_item>::value && !arm->nowait && !sh.chain && !g_dl.cfg.armed_blocks && sh.block_threads == 512u &&
            n <= (size_t)list_cap<Item>::big && armed_grid(t8, 512u, true) <= arm->direct_max) {
            // ... and where the larger tiles do not leave a few workgroups with a quarter more rows than before (over fifteen
            // ranks, 132 919 bytes per rank: 3 tiles of 16 KiB at most instead of 4 of 8, 20.7 us with eight, 21.6 with sixteen),
            // nor many passes of unaligned loads (over eight, 1 500 003 bytes 40.2 : 44.7; over twelve, 1 MiB 61.5 : 53.1), nor in a
            // short list with five destinations and more, where the stores set the pace (from four tiles of 16 KiB a workgroup,
            // eight ranks, 80 / 130 / 200 MiB moved 22.2 / 28.1 / 36.8 : 23.6 / 29.8 / 39.5; five to eight ranks of 1.1 to 3.5 MiB, one or three
            // buffer sets, 1 to 6 % slower on average, the call counted; with the kernel resident before the doorbell rings
            // five ranks 3 to 5 % faster with sixteen, six to eight from 9 % faster to 7 slower by size, within 2.5 on average.  Two to four
            // ranks gain 2 to 17 %, and so do longer lists, whose rows take more finding: nine ranks 6 to 12)
            uint64_t t16 = 0;
            for (size_t i = 0; i < n; ++i) t16 += dl_item_tiles(items[i], 16384);
            const uint64_t g = armed_grid(t8, 512u, true), most8 = (t8 + g - 1) / g, most16 = (t16 + g - 1) / g;
            if (t8 > g && 8u * most16 <= 5u * most8 && (t16 <= 4u * g || ((kmax <= 4u || n > (size_t)NMAX_SMALL) && all_on_grid(items, n)))) {
                sh.tile_bytes = 16384;
                sh.block_threads = 1024;
            }
        }
    }

    if constexpr (std::is_same<Item, dl_plain_item>::value) {
        // Copies off the grid, below the sizes that stream.  Rows next to each other share the lines that their unaligned
        // loads and partly written ends lie in.  Up to 48 MiB moved eight rows to a workgroup, so that they meet in one compute
        // unit: all-to-all, one buffer set / three / sets that fit no cache, 256 threads : 512, 5 ranks of 500 003 bytes (25 MB moved)
        // 3.73 / 4.89 / 7.55 : 3.62 / 4.79 / 7.34 us, 12 of 140 001 5.88 / 7.50 / 10.3 : 5.13 / 7.26 / 10.1, 8 of 300 007 4.72 / 7.08 /
        // 9.94 : 4.64 / 6.94 / 9.85; by how the last tile of a copy falls 16 of 90 001 5.70 / 8.30 / 11.1 : 5.82 / 8.29 / 10.7, 20 of
        // 60 003 6.02 / 8.69 / 11.9 : 6.73 / 8.60 / 11.4.  Beyond, where workgroups are one wavefront, an eighth of the copy to every
        // XCD, so that they meet in one L2; 512 threads have the better figures while all is in the caches, and lose to what was there
        // before where nothing is.  Rows in turn : 512 threads : eighths, 8 of 420 001 7.82 / 9.52 / 11.5 : 6.20 / 8.95 / 12.3 : 7.58 /
        // 9.09 / 11.4, 8 of 524 291 10.7 / 11.2 / 13.5 : 9.1 / 10.7 / 14.1 : 10.7 / 10.9 / 13.4, 15 of 164 228 12.8 / 13.4 / 15.4 : 10.8 /
        // 11.8 / 15.7 : 10.8 / 12.1 / 14.6, 10 of 400 009 13.0 / 13.4 / 15.7 : 12.5 / 13.1 / 16.1 : 11.5 / 12.7 / 15.4, 2 of 9 000 001 11.5 / 11.7 /
        // 14.2 : 11.2 / 11.7 / 14.9 : 10.9 / 11.2 / 14.1.  (Cold sets do not want more loads in flight: two rows per wavefront 7.0 / 9.4 / 13.4
        // for the first of these; nor 512 threads with rows in turn, 7.3 / 9.5 / 12.9, or in eighths, 6.9 / 9.4 / 12.2; nor 128 or 256 in
        // eighths, 6.8 / 9.0 / 12.0 and 6.7 / 9.0 / 12.2, 15 of 164 228 12.3 / 12.7 / 14.7 and 12.2 / 12.3 / 15.4.  Larger ones in turn, as any
        // list: 8 of 2 MiB and 3 bytes.)
        if (free_shape && sh.policy == DL_POL_WT && 2u * total >= OFF_GRID_MIN_BYTES && biggest >= 8192u && !all_on_grid(items, n)) {
            if (sh.block_threads == 64u) {
                sh.eighths = true;
            } else {
                sh.block_threads = 512u;
                sh.tile_bytes = 8192u;
            }
        }
    }
    constexpr int NBIG = list_cap<Item>::big;
    if (n <= (size_t)NBIG) {
        uint64_t tile_end[NBIG];
        if constexpr (std::is_same<Item, dl_fused_item>::value) {
            const uint64_t moved = total * (1ull + kmax);
            if (free_shape && sh.policy == DL_POL_STREAM_OUT) {  // the output outgrows the caches
                uint64_t acc = 0;
                for (size_t i = 0; i < n; ++i) tile_end[i] = acc += dl_pair_blocks(items[i]);
                if (acc < (1ull << 26)) {  // a grid has fewer than 2^32 threads
                    sh.pairs = true;
                    *launched = true;
                    if (n <= (size_t)NMAX_SMALL) return launch_klist<Item, NMAX_SMALL>(items, n, tile_end, sh, stream, arm);
                    return launch_klist<Item, NBIG>(items, n, tile_end, sh, stream, arm);
                }
            } else if (free_shape && sh.policy == DL_POL_WT && moved > FAN_WAVE_MIN_BYTES) {
                // Between the launch-bound requests and those: one wavefront per row, which stores it to all
                // destinations, instead of several that each load it.  Buffers warm / cold, several wavefronts
                // against one, in a graph of 30: all-gather over eight ranks of 32 KiB 1.98 / 1.86 against 2.08 / 1.96 us,
                // 64 KiB 2.42 / 3.36 : 2.19 / 3.12, 256 KiB 4.11 / 5.94 : 3.77 / 4.71, 1 MiB 10.8 / 16.5 : 10.6 / 15.0;
                // 2 MiB to seven others 3.86 / 5.38 : 3.51 / 4.52; of 1 MiB and 5 bytes over five ranks 5.95 / 9.15 : 5.36 / 8.11.
                // A workgroup is that one wavefront, or eight where loads are shifted (1 MiB + 5 over eight
                // ranks: 11.6 us with one, 11.4 with eight, 13.0 with four; 1 MiB: 10.7, 10.6, 11.3).
                const bool on_grid = all_on_grid(items, n);
                sh.split = 1;
                sh.block_threads = on_grid ? 64u : 512u;
                sh.tile_bytes = 16u * sh.block_threads;
                // With one load per row the loads can be streaming ones (see DL_POL_STREAM_IN).  What they give depends on
                // what the calls before left in the Infinity Cache, which a request does not tell: buffers that all fit it, or
                // far exceed it, see no difference; a few sets that together are about its size do.  Over eight / five / two ranks,
                // write-through stores alone : streaming loads as well, 96 MiB moved, one buffer set 11.9 : 12.0, 11.3 :
                // 11.3, 11.9 : 15.2 us, two in turn 12.0 : 12.4, 12.5 : 17.2, 12.9 : 13.8, three 16.0 : 16.2, 16.7 : 15.2,
                // 15.5 : 14.0, eight 19.9 : 20.0, 19.2 : 19.2, 18.3 : 17.5; 128 MiB, two 15.5 : 15.6, 21.3 : 20.3, 19.4 : 17.4,
                // three 25.7 : 24.6, 25.0 : 23.6, 23.6 : 18.8.  The line is where three sets in turn begin to gain (88 MiB
                // over five ranks 16.1 : 14.9, 80 MiB 13.6 : 13.8 and over eight 10.5 : 13.1).
                if (moved >= DL_FAN_STREAM_IN_MIN_BYTES) sh.policy = DL_POL_STREAM_IN;
            }
        }
        const auto count_tiles = [&] {
            for (;;) {
                uint64_t acc = 0;
                for (size_t i = 0; i < n; ++i) {
                    acc += dl_item_tiles(items[i], sh.tile_bytes);
                    tile_end[i] = acc;
                }
                if (acc < (1ull << 30)) break;
                sh.tile_bytes *= 2;  // keep the grid inside the launch limit
            }
        };
        count_tiles();
        // row path: a short list (found by a few scalar compares; bisecting a long one per wavefront
        // measured slower than the general path) and a tile that is exactly one 1 KiB row per
        // wavefront of a sub-group
        // ... or, armed, a list of any length, where few wavefronts are in flight: a waiting kernel, whose grid is capped
        // (all-to-all of 128 / 512 KiB chunks between eight ranks, trigger to done and the call: 21.9 / 44.4 us on the general
        // path, 19.6 / 35.4 this way; all-gather of 480 KiB over 16 ranks 54.8 : 45.7), and a short request without a
        // doorbell (64 chunks of 16 KiB 15.3 : 14.7; with a full grid and 64 MiB moved 25.4 : 25.6, 138 MB 40.8 : 41.6)
        const bool armed_rows = arm && ((!arm->nowait && !sh.chain) || total * (1ull + kmax) <= ARMED_ROWS_MAX_BYTES);
        sh.rows = (n <= (size_t)NMAX_SMALL || armed_rows) && sh.tile_bytes == 16u * (sh.block_threads / sh.split) &&
                  !(sh.max_blocks && !arm);
        // ... or, one-shot, a longer list item by item on a two-dimensional grid (see dl_exec_rows2d_kernel), unless too many of
        // its workgroups find nothing to do: a fifth of them; for plain copies and swaps below the sizes that stream, in
        // workgroups of four rows, three fifths, or whatever a grid of RAGGED_GRID workgroups holds.  Chunks of a
        // mixture-of-experts exchange between eight ranks, three buffer sets in turn, one tile after the other with a search : item by
        // item: 16 tokens per rank of 4 KiB 2.80 : 2.52 us, 24 of 8 KiB 5.73 : 4.83, 24 of 14 KiB 8.8 : 8.0 (sets that
        // fit no cache 11.8 : 10.4), 40 of 10 KiB 9.5 : 9.3, one buffer set 7.8 : 6.6.  Lengths drawn from 1 byte to
        // 40 000: 12 / 30 / 64 copies 2.48 : 2.25, 2.60 : 2.46, 2.67 : 2.64; to 256 KiB (a grid of 2048 / 4096) 32 / 64
        // copies 2.56 : 2.81, 2.74 : 3.35.
        if ((n > (size_t)NMAX_SMALL || sh.eighths) && !arm && !sh.max_blocks) {
            const auto grid_if_even = [&](uint64_t spare) -> uint64_t {  // workgroups of the grid, if `spare` is enough; else 0
                uint64_t widest = 0;
                for (size_t i = 0; i < n; ++i) {
                    const uint64_t t = i ? tile_end[i] - tile_end[i - 1] : tile_end[0];
                    if (t > widest) widest = t;
                }
                return widest * n <= tile_end[n - 1] + spare && widest < (1ull << 31) ? widest * n : 0;
            };
            uint64_t grid = 0;
            if (sh.tile_bytes == 16u * (sh.block_threads / sh.split)) grid = grid_if_even(tile_end[n - 1] / 4);
            if constexpr (!std::is_same<Item, dl_fused_item>::value) {
                if (!grid && n > (size_t)NMAX_SMALL && free_shape && sh.policy == DL_POL_WT) {
                    const dl_launch_shape before = sh;
                    if (sh.block_threads == 64u && biggest >= 4096u) sh.block_threads = 256u;
                    sh.tile_bytes = 16u * sh.block_threads;
                    count_tiles();
                    const uint64_t tiles = tile_end[n - 1];
                    grid = grid_if_even(std::max(tiles + tiles / 2, RAGGED_GRID > tiles ? RAGGED_GRID - tiles : 0));
                    if (!grid) {
                        sh = before;
                        count_tiles();
                    }
                }
            }
            if (grid) {
                sh.rows = true;
                sh.rows2d_width = (uint32_t)(grid / n);
                if (sh.block_threads != 64u) sh.eighths = false;
            }
        }
        if constexpr (!std::is_same<Item, dl_fused_item>::value) {
            // Few workgroups have few loads in flight, and a streaming load takes longer to come back: all-to-all between eight
            // ranks, 2 MiB chunks, 128 / 512 workgroups, one buffer set / three in turn 171 / 240 and 57 / 77 us, with
            // streaming loads 259 / 260 and 79 / 80; with 2048 they are ahead again (50 : 44 with three).
            if (!arm && sh.policy == DL_POL_STREAM_IN && sh.max_blocks && sh.max_blocks < 1024u && tile_end[n - 1] > sh.max_blocks &&
                2u * total < STREAM_BOTH_MIN_BYTES)
                sh.policy = 2u * total <= g_dl.cfg.write_through_max_bytes ? DL_POL_WT : DL_POL_PLAIN;
            if (!arm && sh.policy == DL_POL_STREAM_IN) {
                sh.policy = plain_policy<Item>(sh.policy, sh.rows, all_aligned(items, n), 2u * total);
                if (sh.policy == DL_POL_STREAM && sh.block_threads == 64u && sh.tile_bytes == 1024u) {
                    // (four wavefronts: 88.3 / 174 us at 518 / 1036 MiB moved, one 90.3 / 178)
                    sh.block_threads = 256u;
                    sh.tile_bytes = 4096u;
                    count_tiles();
                }
            }
        }
        *launched = true;
        if (n <= (size_t)NMAX_SMALL) return launch_klist<Item, NMAX_SMALL>(items, n, tile_end, sh, stream, arm);
        return launch_klist<Item, NBIG>(items, n, tile_end, sh, stream, arm);
    }
    *launched = true;
    if constexpr (!std::is_same<Item, dl_fused_item>::value) {
        int rc = DL_OK;
        if (!arm && launch_offsets(items, n, sh, stream, &rc)) return rc;
    }
    return launch_table(items, n, sh, stream, arm);
}

uint32_t floor_pow2(uint64_t v)
{
    uint32_t p = 1;
    while ((uint64_t)p * 2 <= v && p < (1u << 30)) p *= 2;
    return p;
}

}  // namespace

// Tile, workgroup size and fan split for a request.  The finest cut wins: every wavefront moves one 1 KiB row with
// one 16-byte load per lane; larger tiles and capped grids were slower at every size.  What is chosen here is the
// shape of requests that last as long as a launch does: there a row's stores are shared out, at most two per lane, over
// the four wavefronts of a workgroup (a fan-out of 5..8: 1 KiB tiles; 3..4: 2 KiB tiles and two sub-groups; 1:1
// and 1:2 copies: 4 KiB tiles).  Larger copies with several destinations get their shape where they are launched
// (FAN_WAVE_MIN_BYTES, dl_pair_body), larger plain ones below.
dl_launch_shape dl_choose_shape(uint64_t src_bytes, uint64_t max_item_bytes, uint32_t max_k)
{
    const dl_config &c = g_dl.cfg;
    dl_launch_shape sh;
    uint32_t split = c.fan_split;
    if (split == 0) split = max_k > 4 ? 4u : max_k > 2 ? 2u : 1u;
    if (max_k == 1) split = 1;
    const uint64_t moved = src_bytes * (1ull + max_k);  // upper bound on bytes read + written
    uint32_t tile = c.tile_bytes;
    uint32_t most = 256u;  // threads of a workgroup
    if (max_k == 1 && tile == 0 && c.block_threads == 0) most = dl_plain_threads(moved, c.max_blocks != 0);
    if (tile == 0) tile = 16u * most / split;
    sh.tile_bytes = tile;
    uint32_t bt = c.block_threads;
    if (bt == 0) {
        // threads of one sub-group: enough for the tile (or the largest item if that is smaller)
        const uint64_t span = max_item_bytes < tile ? max_item_bytes : tile;
        uint32_t sub = floor_pow2(span / 16 ? span / 16 : 1);
        if (sub > most / split) sub = most / split;
        if (sub < 64) sub = 64;
        bt = sub * split;
    }
    while (split > 1 && bt / split < 64) split /= 2;  // sub-groups are whole wavefronts
    sh.block_threads = bt;
    sh.split = split;
    sh.max_blocks = c.max_blocks;
    // Above write_through_max_bytes copies with several destinations stream their output (see DL_POL_STREAM_OUT) and are
    // written in pairs.  All-gather over eight ranks, three buffer sets in turn, call alone / call and a kernel that reads all of the
    // output: ordinary stores by four wavefronts per row 2.5 MiB per rank 35.3 / 147 us, 3 MiB 41.1 / 157, 4 MiB 53.4 /
    // 180, 6 MiB 76.7 / 238, 8 MiB 102 / 289; write-through by one 34.9 / 144, 41.1 / 154, 55.2 / 177, 82.4 / 234, 111 /
    // 288; streamed in pairs 26.0 / 150, 30.8 / 160, 43.3 / 184, 62.4 / 224, 80.9 / 264.  So up to some 300 MiB moved the
    // reader pays 2 % of its own time for the quarter that the call gains, and with one buffer set that fits the Infinity Cache
    // the call itself loses (2.5 MiB: 23.7, 20.5 and 27.4 us); above, both gain.
    // Streaming hints on both sides where the caller asks for them.  Streaming loads with write-through stores for
    // lists of plain copies from 96 MiB moved, that is 48 MiB read (see DL_POL_STREAM_IN).  All-to-all between eight ranks,
    // write-through stores alone : streaming loads as well, one buffer set / three / eight in turn: 80 MiB 10.8 : 11.3,
    // 12.9 : 12.1, 15.5 : 14.8 us, 96 MiB 12.7 : 13.1, 16.0 : 14.3, 18.1 : 17.4, 128 MiB 16.8 : 17.5, 23.2 : 18.3, 23.3 :
    // 22.4, 192 MiB 24.1 : 25.6, 33.5 : 30.0, 33.4 : 31.8; 64 MiB 8.8 : 10.0, 9.1 : 10.1, 12.7 : 10.6.  Lists that this does
    // not hold for: see plain_policy.
    const bool plain_stream = max_k == 1 && moved >= c.stream_plain_min_bytes;
    sh.policy = moved >= c.nontemporal_min_bytes ? DL_POL_STREAM
                : plain_stream                   ? DL_POL_STREAM_IN
                : moved <= c.write_through_max_bytes ? DL_POL_WT : max_k == 1 ? DL_POL_PLAIN : DL_POL_STREAM_OUT;
    return sh;
}

int dl_exec_plain(const dl_plain_item *items, size_t n, hipStream_t stream, const dl_arm *arm, bool *launched)
{
    return exec_list(items, n, stream, arm, launched);
}
int dl_exec_fused(const dl_fused_item *items, size_t n, hipStream_t stream, const dl_arm *arm, bool *launched)
{
    return exec_list(items, n, stream, arm, launched);
}
int dl_exec_swap(const dl_swap_item *items, size_t n, hipStream_t stream, const dl_arm *arm, bool *launched)
{
    return exec_list(items, n, stream, arm, launched);
}

template <class Item, int NMAX, class Get>
uint64_t standby_list(dl_klist<Item, NMAX> &l, size_t n, uint32_t max_tiles, Get get)
{
    uint64_t acc = 0;
    for (size_t i = 0; i < (size_t)NMAX; ++i) {
        if (i < n) {
            const Item it = get(i);
            acc += dl_item_tiles(it, DL_STANDBY_TILE);
            if (acc > max_tiles) return 0;  // one tile per workgroup, one pass
            l.item[i] = it;
        }
        l.tile_end[i] = i < n ? (uint32_t)acc : 0xFFFFFFFFu;
    }
    l.n = (uint32_t)n;
    l.tile_bytes = DL_STANDBY_TILE;
    l.split = 1;
    l.split_log2 = 0;
    l.wpg_log2 = log2u(DL_STANDBY_THREADS / 64u);
    return acc;
}

uint32_t dl_standby_fill(void *rec_mem, const dl_plan_item *items, size_t n, uint64_t activation, uint64_t ticket,
                         uint64_t *done, uint32_t max_tiles)
{
    const dl_config &c = g_dl.cfg;
    if (n == 0 || n > 64 || c.tile_bytes || c.block_threads || c.max_blocks || c.armed_blocks) return 0;
    static_assert(sizeof(dl_plan_item) == sizeof(dl_fused_item), "plan items are fused items");
    const dl_fused_item *it = reinterpret_cast<const dl_fused_item *>(items);
    static dl_standby_rec r;  // 2 KiB: not on the stack of every call
    uint64_t acc, used;
    if (n <= 8) {
        r.plain = 0;
        acc = standby_list(r.list, n, max_tiles, [&](size_t i) { return it[i]; });
        used = offsetof(dl_standby_rec, list) + sizeof r.list;
    } else {
        for (size_t i = 0; i < n; ++i)
            if (it[i].k != 1) return 0;
        r.plain = 1;
        acc = standby_list(r.copies, n, max_tiles,
                           [&](size_t i) { return dl_plain_item{it[i].src, it[i].dst[0], it[i].bytes}; });
        used = offsetof(dl_standby_rec, copies) + sizeof r.copies;
    }
    if (acc == 0) return 0;
    r.ticket_front = r.ticket_back = ticket;
    r.activation = activation;
    r.done = done;
    r.arrivals = 0;
    // The record may live in device memory mapped write-combined: plain 8-byte stores in ascending order, of the
    // part that this kind of list uses and of the closing ticket.
    static uint64_t words[sizeof r / 8];
    memcpy(words, &r, sizeof r);
    volatile uint64_t *out = (volatile uint64_t *)rec_mem;
    for (size_t q = 0; q < (used + 7) / 8; ++q) out[q] = words[q];
    out[sizeof r / 8 - 1] = words[sizeof r / 8 - 1];
    return acc <= DL_DONE_WORDS ? (uint32_t)acc : 1u;
}

int dl_standby_launch(void *rec_mem, const dl_arm *a, hipStream_t stream)
{
    hipLaunchKernelGGL(dl_standby_kernel, dim3(DL_STANDBY_GRID), dim3(DL_STANDBY_THREADS), 0, stream,
                       (dl_standby_rec *)rec_mem, *a);
    DL_HIP(hipGetLastError());
    return DL_OK;
}

int dl_launch_plain_table(const dl_plain_item *dev_items, uint32_t m, uint32_t entry_bytes, uint64_t moved, bool aligned,
                          hipStream_t stream)
{
    if (m == 0) return DL_OK;
    const int policy = plain_policy<dl_plain_item>(dl_choose_shape(moved / 2, entry_bytes, 1).policy, false, aligned, moved);
    dl_with_policy(policy, [&](auto pol) {
        hipLaunchKernelGGL((dl_exec_table_kernel<dl_plain_item, decltype(pol)::value, false>), dim3(m), dim3(256), 0,
                           stream, dev_items, m, 1u, dl_push_kernel_args(0));
    });
    DL_HIP(hipGetLastError());
    return DL_OK;
}

void *dl_scratch_acquire(size_t *slot)
{
    if (!g_ring.base) return nullptr;
    const size_t s = g_ring.next % RING_SLOTS;
    if (g_ring.used[s] && wait_for_readers(g_ring.ev[s], g_ring.armed[s]) != DL_OK) return nullptr;
    ++g_ring.next;
    g_ring.armed[s] = 0;
    *slot = s;
    return g_ring.dev + s * RING_SLOT_BYTES;
}

int dl_scratch_release(size_t slot, hipStream_t stream)
{
    DL_HIP(hipEventRecord(g_ring.ev[slot], stream));
    g_ring.used[slot] = true;
    return DL_OK;
}

void dl_ring_forget_armed()
{
    for (size_t s = 0; s < RING_SLOTS; ++s) g_ring.armed[s] = 0;
    for (size_t s = 0; s < PUSH_SLOTS; ++s) g_ring.push_armed[s] = 0;
}

void dl_ring_own_stream(hipStream_t stream)
{
    if (!stream && g_ring.batch_len && g_ring.batch_stream == g_ring.own_stream) (void)push_close_batch();
    g_ring.own_stream = stream;
}

// The device error word: host-coherent memory that a kernel writes when it gives up on a table that never
// became complete (see dl_pushed).  Read, and cleared, by dl_last_device_error().
static uint64_t *g_lost = nullptr;
// Test hook (dl_debug_lose_next_table): the kernel of the next table that goes through the BAR is told a stamp
// that its slot will never hold and this many looks, so that the give-up path runs, every wait still bounded.
static uint32_t g_debug_lose_tries = 0;

dl_pushed dl_push_kernel_args(uint64_t stamp)
{
    dl_pushed ps{stamp, DL_PUSHED_TRIES, 0u, g_lost};
    if (stamp && g_debug_lose_tries) {
        ps.stamp = stamp | (1ull << 62);
        ps.tries = g_debug_lose_tries;
        g_debug_lose_tries = 0;
    }
    return ps;
}

char *dl_push_acquire(size_t bytes, hipStream_t stream, int *rc) { return push_acquire(bytes, stream, rc); }
uint64_t dl_push_seal(char *slot) { return push_seal(slot); }
int dl_push_commit(hipStream_t stream) { return push_commit(stream, 0); }

bool dl_device_error_pending() { return g_lost && __atomic_load_n(g_lost, __ATOMIC_ACQUIRE) != 0; }

extern "C" int dl_last_device_error(void)
{
    if (!g_lost) return DL_OK;
    return __atomic_exchange_n(g_lost, 0ull, __ATOMIC_ACQ_REL) ? DL_ERR_LOST : DL_OK;
}

extern "C" int dl_debug_lose_next_table(uint32_t tries)
{
    if (!g_dl.inited) return DL_ERR_STATE;
    if (!g_ring.push || !g_dl.cfg.table_push) return DL_ERR_STATE;  // no table goes through the BAR here
    if (tries > 1024) return DL_ERR_INVALID;  // 0 disarms the hook
    g_debug_lose_tries = tries;
    return DL_OK;
}

// Device memory that the host can store into: only where one PCIe BAR covers all of the device's memory.  Made
// once per process and kept until it ends.
void *dl_bar_memory(size_t bytes)
{
    const char *off = getenv("DL_NO_BAR");  // "1": keep everything the host writes in host memory
    if (off && off[0] == '1') return nullptr;
    int large_bar = 0;
    if (hipDeviceGetAttribute(&large_bar, hipDeviceAttributeIsLargeBar, g_dl.device) != hipSuccess || large_bar != 1) {
        (void)hipGetLastError();
        return nullptr;
    }
    void *p = nullptr;
    if (hipExtMallocWithFlags(&p, bytes, hipDeviceMallocFinegrained) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    if (hipMemset(p, 0, bytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;  // left allocated and unused
    }
    return p;
}

int dl_exec_init()
{
    // kept for the life of the process, per device: what was made for another device is left behind
    static int push_device = -1;
    static char *push_memory = nullptr;
    if (push_device != g_dl.device) {
        push_device = g_dl.device;
        push_memory = (char *)dl_bar_memory(PUSH_SLOTS * PUSH_SLOT_BYTES);
    }
    if (g_ring.base) return DL_OK;
    g_ring.push = push_memory;
    g_ring.push_next = 0;
    g_ring.batch_len = 0;
    g_ring.own_stream = nullptr;
    for (size_t q = 0; q < PUSH_SLOTS; ++q) {
        DL_HIP(hipEventCreateWithFlags(&g_ring.push_ev[q], hipEventDisableTiming));
        g_ring.push_used[q] = false;
        g_ring.push_cover[q] = -1;
        g_ring.push_armed[q] = 0;
    }
    DL_HIP(hipHostMalloc((void **)&g_lost, 64, hipHostMallocCoherent | hipHostMallocMapped));
    *g_lost = 0;
    g_debug_lose_tries = 0;
    DL_HIP(hipHostMalloc((void **)&g_ring.base, RING_SLOTS * RING_SLOT_BYTES, hipHostMallocDefault));
    DL_HIP(hipMalloc((void **)&g_ring.dev, RING_SLOTS * RING_SLOT_BYTES));
    for (size_t s = 0; s < RING_SLOTS; ++s) {
        DL_HIP(hipEventCreateWithFlags(&g_ring.ev[s], hipEventDisableTiming));
        g_ring.used[s] = false;
    }
    g_ring.next = 0;
    return DL_OK;
}

int dl_exec_shutdown()
{
    if (!g_ring.base) return DL_OK;
    for (size_t s = 0; s < RING_SLOTS; ++s) {
        if (g_ring.used[s]) (void)hipEventSynchronize(g_ring.ev[s]);
        (void)hipEventDestroy(g_ring.ev[s]);
    }
    // everything launched has ended before the tables' memory is handed out again after the next dl_exec_init
    // (the open batch has no event yet; its stream is the default one or the library's, which is gone by now)
    (void)hipDeviceSynchronize();
    for (size_t q = 0; q < PUSH_SLOTS; ++q) (void)hipEventDestroy(g_ring.push_ev[q]);
    (void)hipHostFree(g_ring.base);
    (void)hipFree(g_ring.dev);
    (void)hipHostFree(g_lost);
    g_lost = nullptr;
    g_ring.base = nullptr;
    g_ring.dev = nullptr;
    return DL_OK;
}
