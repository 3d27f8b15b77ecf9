"""GPU parity: every operation, through the C boundary, byte for byte against
the CPU checker on the same seeded inputs.  The bar is bit-exact (pure data
movement), and bytes outside every destination must stay untouched."""

import os

import numpy as np
import pytest

import paper_2511_06605_amd as dl
from paper_2511_06605_amd import inputs
from paper_2511_06605_amd.inputs import KiB, MiB

from gpu_util import DevBuf, stream, sync

pytestmark = pytest.mark.gpu

VALIDATE_ALL = os.environ.get("DL_TEST_VALIDATE") == "1"
FORCED = bool(os.environ.get("DL_TEST_CONFIG")) or VALIDATE_ALL   # settings that send requests other ways


@pytest.fixture(scope="module", autouse=True)
def library():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    dl.dl_init(0)
    base = dl.dl_get_config()
    # DL_TEST_VALIDATE=1 runs every test with the hazard check on: it must refuse none of the valid requests
    dl.dl_set_validate(VALIDATE_ALL)
    # DL_TEST_CONFIG="max_blocks=64,fan_split=1" runs every test with those tunables as the defaults
    forced = dict(kv.split("=") for kv in os.environ.get("DL_TEST_CONFIG", "").split(",") if kv)
    if forced:
        dl.dl_set_config(**{k: int(v) for k, v in forced.items()})
    yield
    dl.dl_set_config(base)
    dl.dl_set_validate(False)
    dl.dl_shutdown()


@pytest.fixture()
def cfg():
    """Set tunables for one test and restore the defaults afterwards."""
    base = dl.dl_get_config()
    saved = {f[0]: getattr(base, f[0]) for f in base._fields_}

    def set_(**kw):
        dl.dl_set_config(**kw)
    yield set_
    dl.dl_set_config(**saved)


def run_allgather(ref, W, B, seed, kind="u8", shifts=None, in_place=False):
    ins = inputs.allgather_inputs(W, B, seed, kind)
    want = ref.allgather(ins)
    shifts = shifts or [0] * (2 * W)
    d_out = [DevBuf(W * B, shift=shifts[W + r]) for r in range(W)]
    if in_place:
        for r in range(W):
            d_out[r].view()[r * B:(r + 1) * B].copy_(__import__("torch").from_numpy(ins[r]))
        in_ptrs = [d_out[r].ptr(r * B) for r in range(W)]
        d_in = []
    else:
        d_in = [DevBuf(B, fill=ins[r], shift=shifts[r]) for r in range(W)]
        in_ptrs = [b.ptr() for b in d_in]
    dl.dl_allgather(in_ptrs, [b.ptr() for b in d_out], B, stream())
    sync()
    for r in range(W):
        assert np.array_equal(d_out[r].host(), want[r]), f"rank {r} differs (W={W}, B={B})"
        assert d_out[r].guards_intact()
    for r, b in enumerate(d_in):
        assert np.array_equal(b.host(), ins[r]) and b.guards_intact()


def run_alltoall(ref, C, seed, kind="u8"):
    W = C.shape[0]
    ins = inputs.alltoall_inputs(C, seed, kind)
    want = ref.alltoall(ins, C)
    d_in = [DevBuf(ins[i].size, fill=ins[i]) for i in range(W)]
    d_out = [DevBuf(want[j].size) for j in range(W)]
    dl.dl_alltoall([b.ptr() for b in d_in], [b.ptr() for b in d_out], C, stream())
    sync()
    for j in range(W):
        assert np.array_equal(d_out[j].host(), want[j]), f"receiver {j} differs"
        assert d_out[j].guards_intact()
    return d_out, ins


# ------------------------------------------------------------------ all-gather

def test_allgather_config0_uint8_64KiB(ref):
    """W = 8, 64 KiB per rank of uniform bytes, seed 0: every bit pattern moves unchanged."""
    run_allgather(ref, 8, 64 * KiB, seed=0)


@pytest.mark.parametrize("B", [1, 15, 16, 17, 255, 4096, 4097, 64 * KiB + 1, 1 * MiB + 3, 3 * MiB])
def test_allgather_sizes_ragged(ref, B):
    run_allgather(ref, 8, B, seed=B, kind="bf16" if B % 2 == 0 else "u8")


@pytest.mark.parametrize("W", [1, 2, 3, 5, 13, 64])
def test_allgather_rank_counts(ref, W):
    run_allgather(ref, W, 5000, seed=W)


@pytest.mark.parametrize("B", [4 * KiB << i for i in range(14)])
def test_allgather_sweep_points_bf16(ref, B):
    """Every point of the all-gather size sweep that the benchmark times, 4 KiB .. 32 MiB per rank, same seeds and
    launch configuration (64 MiB: test_allgather_full_size_64MiB)."""
    run_allgather(ref, 8, B, seed=B.bit_length() - 1, kind="bf16")


@pytest.mark.parametrize("tokens", [1, 8, 32, 128, 256])
def test_allgather_tp_decode(ref, tokens):
    run_allgather(ref, 8, inputs.tp_decode_bytes_per_rank(tokens), seed=tokens, kind="bf16")


def test_allgather_in_place(ref):
    run_allgather(ref, 8, 70001, seed=3, in_place=True)


@pytest.mark.parametrize("case", ["coaligned_odd", "mod4", "mod1"])
def test_allgather_misaligned(ref, case):
    W = 4
    if case == "coaligned_odd":
        shifts = [5] * (2 * W)                       # all equal modulo 16, none aligned
    elif case == "mod4":
        shifts = [0, 4, 8, 12, 0, 4, 8, 12]          # agree modulo 4 only
    else:
        shifts = [0, 1, 2, 3, 7, 9, 11, 13]          # agree modulo 1 only
    # W*B a multiple of 16 keeps slot offsets from changing the residues
    run_allgather(ref, W, 40000, seed=11, shifts=shifts)
    run_allgather(ref, W, 16 * 77, seed=12, shifts=shifts)


def test_allgather_unfused_plain_copies(ref, cfg):
    cfg(fuse_broadcast=0)
    run_allgather(ref, 8, 100000, seed=5)


@pytest.mark.parametrize("tile,block", [(1024, 64), (4096, 256), (65536, 512), (1 << 20, 128)])
def test_allgather_forced_tiles(ref, cfg, tile, block):
    cfg(tile_bytes=tile, block_threads=block)
    run_allgather(ref, 8, 3 * tile + 16 * 5 + 7, seed=tile)
    run_allgather(ref, 3, tile - 16, seed=tile + 1)


@pytest.mark.parametrize("split,block,tile", [(1, 64, 1024), (1, 256, 4096), (2, 128, 1024), (2, 256, 2048),
                                              (4, 256, 1024), (4, 512, 4096), (4, 64, 1024), (2, 512, 65536)])
def test_allgather_forced_fan_split(ref, cfg, split, block, tile):
    """Destinations shared out over sub-groups of a workgroup: every fan-out 1..8 (W ranks, and the
    in-place layout that drops one), ragged sizes, for every split / workgroup / tile combination.
    A workgroup too small for the split (4 over 64 threads) falls back to fewer sub-groups."""
    cfg(fan_split=split, block_threads=block, tile_bytes=tile)
    for W in (1, 2, 3, 4, 5, 6, 7, 8):
        run_allgather(ref, W, 3 * tile + 16 * 3 + 5, seed=100 * split + W)
    run_allgather(ref, 8, 900, seed=split)
    run_allgather(ref, 8, 70001, seed=split + 1, in_place=True)
    run_allgather(ref, 13, 5000, seed=split + 2)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15])
def test_broadcast_default_split_every_fanout(ref, k):
    n = 300 * KiB + 48
    src = inputs.payload(np.random.default_rng(k), n, "bf16")
    d_src = DevBuf(n, fill=src)
    d_dst = [DevBuf(n) for _ in range(k)]
    dl.dl_broadcast(d_src.ptr(), [b.ptr() for b in d_dst], n, stream())
    sync()
    for b, w in zip(d_dst, ref.broadcast(src, k)):
        assert np.array_equal(b.host(), w) and b.guards_intact()


@pytest.mark.parametrize("cap", [1, 7, 64, 4096])
def test_capped_grid_workgroups_stride_over_tiles(ref, cfg, cap):
    """max_blocks caps the one-shot grid; the workgroups then take tiles b, b + grid, ... (general path)."""
    cfg(max_blocks=cap)
    run_allgather(ref, 8, 300 * KiB + 16, seed=cap)
    run_allgather(ref, 3, 70001, seed=cap + 1)
    run_alltoall(ref, inputs.random_chunks(8, 90000, seed=cap, zero_frac=0.2), seed=cap + 2)
    run_batch(ref, 5, 200000, 8 * MiB, seed=cap + 3, align=16)


@pytest.mark.parametrize("wt_max", [0, 1 << 62])
def test_capped_grid_with_the_policies_of_large_lists(ref, cfg, wt_max):
    """The size from which plain lists get streaming loads set to one byte: a capped grid keeps write-through or
    ordinary stores."""
    cfg(max_blocks=33, stream_plain_min_bytes=1, write_through_max_bytes=wt_max)
    run_alltoall(ref, inputs.uniform_chunks(8, 40000), seed=38, kind="u8")
    run_alltoall(ref, inputs.random_chunks(7, 100000, seed=39, zero_frac=0.1), seed=40)
    run_batch(ref, 60, 30001, 32 * MiB, seed=41, align=1)


def test_allgather_nontemporal_path(ref, cfg):
    cfg(nontemporal_min_bytes=0)
    run_allgather(ref, 8, 300001, seed=8)
    cfg(nontemporal_min_bytes=1 << 62)
    run_allgather(ref, 8, 300001, seed=8)


@pytest.mark.parametrize("wt_max", [0, 1 << 62])
def test_store_policy_write_through_on_and_off(ref, cfg, wt_max):
    """Write-through stores forced on / off for every path: row kernels, general path with heads and
    tails, misaligned (narrow elements), long lists (table kernel), 1:1 and fused."""
    cfg(write_through_max_bytes=wt_max)
    run_allgather(ref, 8, 256 * KiB, seed=31, kind="bf16")
    run_allgather(ref, 8, 300001, seed=32)
    run_allgather(ref, 4, 40000, seed=33, shifts=[0, 1, 2, 3, 7, 9, 11, 13])
    run_alltoall(ref, inputs.uniform_chunks(8, 64 * KiB), seed=34, kind="fp16")
    run_alltoall(ref, inputs.random_chunks(16, 100000, seed=35, zero_frac=0.1), seed=36)
    run_batch(ref, 200, 50000, 64 * MiB, seed=37, align=16)


def test_allgather_full_size_64MiB(ref):
    """Largest sweep point, default launch configuration: 0.5 GiB in, 4 GiB out."""
    import torch
    W, B = 8, 64 * MiB
    ins = inputs.allgather_inputs(W, B, seed=26, kind="bf16")
    d_in = [torch.from_numpy(a).cuda() for a in ins]
    d_out = [torch.full((W * B,), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(W)]
    dl.dl_allgather(d_in, d_out, B, stream())
    sync()
    want = ref.allgather(ins)
    for r in range(W):
        assert np.array_equal(d_out[r].cpu().numpy(), want[r]), f"rank {r}"


# ------------------------------------------------------------------ all-to-all

@pytest.mark.parametrize("c", [1 * KiB << i for i in range(13)])
def test_alltoall_uniform_fp16(ref, c):
    """Every point of the all-to-all sweep, 1 KiB .. 4 MiB per pair, as the benchmark draws it."""
    run_alltoall(ref, inputs.uniform_chunks(8, c), seed=c.bit_length(), kind="fp16")


@pytest.mark.parametrize("W,seed", [(2, 0), (3, 1), (8, 2), (8, 3), (13, 4)])
def test_alltoall_nonsymmetric_with_zero_chunks(ref, W, seed):
    C = inputs.random_chunks(W, 50000, seed=seed, zero_frac=0.25)
    assert W == 1 or not np.array_equal(C, C.T)
    run_alltoall(ref, C, seed=seed + 50)


def test_alltoall_twice_is_identity_on_gpu(ref):
    C = inputs.random_chunks(8, 30000, seed=9, zero_frac=0.2, multiple_of=16)
    d_mid, ins = run_alltoall(ref, C, seed=10)
    d_back = [DevBuf(ins[i].size) for i in range(8)]
    dl.dl_alltoall([b.ptr() for b in d_mid], [b.ptr() for b in d_back], C.T, stream())
    sync()
    for i in range(8):
        assert np.array_equal(d_back[i].host(), ins[i])


@pytest.mark.parametrize("T", [16, 128, 512])
def test_alltoall_moe_dispatch(ref, T):
    C = inputs.moe_dispatch_chunks(8, T, seed=T)
    assert int(C.sum()) == 8 * 8 * T * 14336
    run_alltoall(ref, C, seed=T + 1, kind="bf16")


def test_alltoall_moe_dispatch_skewed(ref):
    run_alltoall(ref, inputs.moe_dispatch_chunks(8, 128, seed=7, skew_alpha=0.5), seed=8, kind="bf16")


def test_alltoall_many_ranks_long_list(ref):
    """W = 16 gives 256 copies: more than the kernel-argument list holds."""
    C = inputs.random_chunks(16, 200000, seed=21, zero_frac=0.1)
    run_alltoall(ref, C, seed=22)


# ------------------------------------------------------------------- broadcast

@pytest.mark.parametrize("k,n,kind", [(7, 2 * MiB, "bf16"), (1, 12345, "u8"), (8, 4096, "u8"), (9, 100001, "u8"),
                                      (20, 77777, "u8"), (64, 1000, "u8")])
def test_broadcast(ref, k, n, kind):
    src = inputs.payload(np.random.default_rng(k * 7 + n), n, kind)
    want = ref.broadcast(src, k)
    d_src = DevBuf(n, fill=src)
    d_dst = [DevBuf(n) for _ in range(k)]
    dl.dl_broadcast(d_src.ptr(), [b.ptr() for b in d_dst], n, stream())
    sync()
    for b, w in zip(d_dst, want):
        assert np.array_equal(b.host(), w) and b.guards_intact()
    assert np.array_equal(d_src.host(), src)


# --------------------------------------------------------------- batched copies

def run_batch(ref, n, copy_bytes, arena_bytes, seed, align=256):
    arena, descs = inputs.b2b_batch(n, copy_bytes, arena_bytes, seed, align)
    want = ref.batch_copy([arena.copy()], [(0, s, 0, d, nb) for s, d, nb in descs])[0]
    d = DevBuf(arena_bytes, fill=arena)
    dl.dl_batch_copy([(d.ptr(int(s)), d.ptr(int(t)), int(nb)) for s, t, nb in descs], stream())
    sync()
    assert np.array_equal(d.host(), want)
    assert d.guards_intact()


def test_batch_config3_64_copies_of_16KiB(ref):
    run_batch(ref, 64, 16 * KiB, 64 * MiB, seed=3)


@pytest.mark.parametrize("n,nb,arena,align", [(1, 100, 4096, 1), (5, 1000, 64 * KiB, 8), (65, 5000, 4 * MiB, 16),
                                              (1000, 4096, 32 * MiB, 256), (300, 70001, 128 * MiB, 1)])
def test_batch_shapes(ref, n, nb, arena, align):
    run_batch(ref, n, nb, arena, seed=n, align=align)


@pytest.mark.parametrize("n,max_bytes,shared", [(7, 3000, 0.0), (40, 200000, 0.0), (64, 70000, 0.5), (300, 40000, 0.3),
                                                (2000, 9000, 0.0)])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_batch_of_unequal_sizes_and_alignments(ref, n, max_bytes, shared, seed):
    """One list mixing 16-, 4- and 1-byte element paths, heads, tails, empty copies and shared sources."""
    arena, descs = inputs.mixed_batch(n, max_bytes, 48 * MiB, seed=1000 * seed + n, shared_sources=shared)
    want = ref.batch_copy([arena.copy()], [(0, s, 0, d, nb) for s, d, nb in descs])[0]
    d = DevBuf(arena.size, fill=arena)
    dl.dl_batch_copy([(d.ptr(int(s)), d.ptr(int(t)), int(nb)) for s, t, nb in descs], stream())
    sync()
    assert np.array_equal(d.host(), want)
    assert d.guards_intact()


def test_batch_long_list_with_large_items(ref, cfg):
    """More copies than the argument list holds, each several tiles long."""
    cfg(tile_bytes=4096)
    run_batch(ref, 200, 50000, 64 * MiB, seed=77, align=16)


def test_batch_kv_fetch_shape(ref):
    """256 dispersed block copies in one batch, as a paged KV-cache fetch issues them."""
    run_batch(ref, 256, 128 * KiB, 256 * MiB, seed=5)


# ------------------------------------------- token dispatch, fan-out batches, broadcast inference

def run_token_dispatch(ref, W, counts, row, seed, kind="u8", drop=None, skew=None, experts=256, top_k=8):
    ins = inputs.token_rows(W, counts, row, seed=seed, kind=kind)
    dest = inputs.moe_token_destinations(W, counts, seed=seed + 1, n_experts=experts, top_k=top_k, skew_alpha=skew)
    if drop:
        dest[::drop] = 0
    want = ref.token_dispatch(ins, row, dest)
    d_in = [DevBuf(a.size, fill=a) for a in ins]
    d_out = [DevBuf(w.size) for w in want]
    tok = [counts] * W if np.isscalar(counts) else counts
    dl.dl_token_dispatch([b.ptr() for b in d_in], [b.ptr() for b in d_out], tok, row, dest, stream())
    sync()
    for j in range(W):
        assert np.array_equal(d_out[j].host(), want[j]), f"receiver {j} differs"
        assert d_out[j].guards_intact()
    return int(dest.sum())


@pytest.mark.parametrize("T", [16, 128, 512])
def test_token_dispatch_moe_hidden_7168_bf16_top8(ref, T):
    """W = 8, 256 experts split 32 per rank, top-8: thousands of 14 KiB rows, each to 1..8 ranks."""
    copies = run_token_dispatch(ref, 8, T, 14336, seed=T, kind="bf16")
    assert 8 * T <= copies <= 8 * 8 * T


@pytest.mark.parametrize("W,counts,row,drop", [(1, [5], 1000, None), (3, [7, 0, 2], 100, 3), (8, [1] * 8, 17, None),
                                               (5, [40, 3, 0, 11, 9], 4097, 4), (13, [6] * 13, 5000, 5)])
def test_token_dispatch_ragged(ref, W, counts, row, drop):
    run_token_dispatch(ref, W, counts, row, seed=W * 7 + row, drop=drop, experts=16 * W, top_k=min(8, W))


@pytest.mark.parametrize("device_lowering,push", [(0, 1), (1, 1), (0, 0), (1, 0)])
@pytest.mark.parametrize("W,counts,row,drop", [(8, 100, 14336, None), (8, [300, 0, 5, 700, 64, 0, 1, 90], 1040, 3),
                                               (3, [400, 1, 200], 48, 5), (1, [600], 4096, 4),
                                               (5, [0, 0, 513, 0, 0], 2048 + 16, None), (8, 2000, 256, 7)])
def test_token_dispatch_lowered_on_device_and_on_host(ref, cfg, device_lowering, push, W, counts, row, drop):
    """With 8 ranks, 512 tokens or more and aligned rows the copy list is built on the device from the mask;
    the host lowering of the same request must give the same bytes.  Empty ranks, tokens without
    destination, rows shorter than one tile; other rank counts (host lowering either way).  Mask or table
    written through the BAR, or through the pinned ring."""
    cfg(device_lowering=device_lowering, table_push=push)
    run_token_dispatch(ref, W, counts, row, seed=W + row, drop=drop, experts=32 * W, top_k=min(8, W))


@pytest.mark.parametrize("counts,row,top_k,mask_value", [
    ([64] * 8, 16, 8, 1),                       # exactly the smallest request the device lowering takes
    ([63] * 7 + [70], 32, 8, 255),              # 511: just below it; mask bytes other than 1
    ([1363] * 8, 16, 2, 1),                     # 10 904 tokens: the most whose mask and table fit the staging slot
    ([1364] * 8, 16, 2, 1),                     # 10 912: just above
    ([8160] * 8, 16, 2, 1),                     # 65 280: far above
    ([1000] * 8, 32, 3, 1),                     # 8000: about the longest mask that goes through the BAR
    ([1030] * 8, 32, 3, 1),                     # 8240: just too long for that
    ([700, 1, 0, 300, 0, 0, 29, 2], 1024, 1, 2),     # every token to exactly one rank
    ([100] * 8, 2048, 64, 7),                   # (nearly) every token to all eight ranks
    ([257, 255, 256, 1, 0, 511, 64, 63], 1040, 3, 1),  # rank boundaries off the builder's 256-token blocks
    ([300] * 8, 64, 4, 0x80),                   # mask bytes whose only set bit is the highest
    ([300] * 8, 64, 4, 0x10),
])
def test_token_dispatch_device_lowering_edges(ref, counts, row, top_k, mask_value):
    W = 8
    ins = inputs.token_rows(W, counts, row, seed=sum(counts) + row, kind="u8")
    dest = inputs.moe_token_destinations(W, counts, seed=top_k + row, n_experts=256, top_k=top_k) * np.uint8(mask_value)
    want = ref.token_dispatch(ins, row, dest)
    d_in = [DevBuf(a.size, fill=a) for a in ins]
    d_out = [DevBuf(w.size) for w in want]
    dl.dl_token_dispatch([b.ptr() for b in d_in], [b.ptr() for b in d_out], counts, row, dest, stream())
    sync()
    for j in range(W):
        assert np.array_equal(d_out[j].host(), want[j]), f"receiver {j} differs"
        assert d_out[j].guards_intact()


def test_token_dispatch_skewed_experts(ref):
    run_token_dispatch(ref, 8, 128, 14336, seed=21, kind="bf16", skew=0.3)


def test_batch_fanout_mixed_items(ref):
    """Read-once/write-k items with every k in one batch, ragged sizes; checked as the plain copies they stand for."""
    rng = np.random.default_rng(8)
    n_items, slot = 24, 20000
    arena = rng.integers(0, 256, (n_items * 9 + 1) * slot, dtype=np.uint8)
    d = DevBuf(arena.size, fill=arena)
    items, copies = [], []
    for i in range(n_items):
        k, nb = 1 + i % 8, int(rng.integers(1, slot))
        s = i * 9 * slot
        dsts = [s + (q + 1) * slot for q in range(k)]
        items.append(dict(src=d.ptr(s), bytes=nb, dst=[d.ptr(t) for t in dsts]))
        copies += [(0, s, 0, t, nb) for t in dsts]
    want = ref.batch_copy([arena.copy()], copies)[0]
    dl.dl_batch_fanout(items, stream())
    sync()
    assert np.array_equal(d.host(), want) and d.guards_intact()


def in_chunks(ref, arena, copies, chunk=4000):
    """The checker on a long list whose sources lie in a part of the arena that no copy writes: applied a few
    thousand copies at a time (its hazard check compares all pairs), which gives what the whole batch gives."""
    for i in range(0, len(copies), chunk):
        ref.batch_copy([arena], copies[i:i + chunk])
    return arena


def test_lists_longer_than_one_staging_slot(ref):
    """45 000 plain copies and 13 000 read-once/write-2 copies: more table entries than one slot of the staging
    ring holds, so each request takes several table kernels.  Ragged sizes below one row, offsets on 80-byte
    slots (every alignment)."""
    rng = np.random.default_rng(12)
    n, slot = 45000, 80
    arena = rng.integers(0, 256, 2 * n * slot, dtype=np.uint8)
    d = DevBuf(arena.size, fill=arena)
    src = rng.integers(0, n, n) * slot + rng.integers(0, 8, n)
    dst = (n + rng.permutation(n)) * slot + rng.integers(0, 8, n)
    nb = rng.integers(1, slot - 8, n)
    want = in_chunks(ref, arena.copy(), [(0, s, 0, t, m) for s, t, m in zip(src, dst, nb)])
    dl.dl_batch_copy([(d.ptr(int(s)), d.ptr(int(t)), int(m)) for s, t, m in zip(src, dst, nb)], stream())
    sync()
    assert np.array_equal(d.host(), want) and d.guards_intact()

    n = 13000
    arena = rng.integers(0, 256, 3 * n * slot, dtype=np.uint8)
    d = DevBuf(arena.size, fill=arena)
    src = rng.integers(0, n, n) * slot
    perm = rng.permutation(2 * n)
    nb = rng.integers(1, slot + 1, n)
    items, copies = [], []
    for i in range(n):
        t0, t1 = (n + int(perm[2 * i])) * slot, (n + int(perm[2 * i + 1])) * slot
        items.append(dict(src=d.ptr(int(src[i])), bytes=int(nb[i]), dst=[d.ptr(t0), d.ptr(t1)]))
        copies += [(0, int(src[i]), 0, t0, int(nb[i])), (0, int(src[i]), 0, t1, int(nb[i]))]
    want = in_chunks(ref, arena.copy(), copies)
    dl.dl_batch_fanout(items, stream())
    sync()
    assert np.array_equal(d.host(), want) and d.guards_intact()


@pytest.mark.parametrize("push", [1, 0])
def test_many_table_requests_in_flight_on_changing_streams(ref, cfg, push):
    """220 requests of 70 to 400 copies each (more than fit the kernel arguments: every request writes a table),
    issued back to back without any synchronisation between them, on three streams that take turns every few
    requests, each request on buffers of its own (one in ten with equal copies of 16 KiB: the row kernel over a
    table of whole items).  The table memory is reused several times over while earlier
    requests may still be running, so a table overwritten too early or read stale shows as a wrong byte."""
    import torch
    cfg(table_push=push)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    rng = np.random.default_rng(77)
    cases = []
    for r in range(220):
        n, slot = int(rng.integers(70, 400)), int(rng.choice([48, 512, 2048, 16384], p=[0.3, 0.3, 0.3, 0.1]))
        arena = rng.integers(0, 256, 2 * n * slot, dtype=np.uint8)
        src = rng.integers(0, n, n) * slot + (rng.integers(0, 4, n) if slot == 48 else 0)
        dst = (n + rng.permutation(n)) * slot
        nb = rng.integers(1, slot - 4, n) if slot == 48 else np.full(n, slot if r % 3 else slot - 16)
        copies = [(int(a), int(b), int(m)) for a, b, m in zip(src, dst, nb)]
        cases.append((arena, DevBuf(arena.size, fill=arena), copies))
    torch.cuda.synchronize()
    for r, (arena, d, copies) in enumerate(cases):
        st = streams[(r // 5) % 3 if r % 40 < 25 else 0]
        dl.dl_batch_copy([(d.ptr(a), d.ptr(b), m) for a, b, m in copies], st)
    torch.cuda.synchronize()
    for r, (arena, d, copies) in enumerate(cases):
        want = ref.batch_copy([arena.copy()], [(0, a, 0, b, m) for a, b, m in copies])[0]
        assert np.array_equal(d.host(), want) and d.guards_intact(), f"request {r}"


@pytest.mark.parametrize("infer", [0, 1])
def test_batch_copy_with_and_without_broadcast_inference(ref, cfg, infer):
    """An all-gather written as 64 plain copies (receiver-major), plus unrelated copies: same bytes either way."""
    cfg(infer_broadcast=infer)
    W, B = 8, 50000
    ins = inputs.allgather_inputs(W, B, seed=6)
    want = ref.allgather(ins)
    d_in = [DevBuf(B, fill=a) for a in ins]
    d_out = [DevBuf(W * B) for _ in range(W)]
    extra_src = DevBuf(3000, fill=inputs.payload(np.random.default_rng(1), 3000))
    extra_dst = DevBuf(3000)
    descs = [(d_in[j].ptr(), d_out[r].ptr(j * B), B) for r in range(W) for j in range(W)]
    descs += [(extra_src.ptr(0), extra_dst.ptr(0), 1500), (extra_src.ptr(1500), extra_dst.ptr(1500), 1500)]
    dl.dl_batch_copy(descs, stream())
    sync()
    for r in range(W):
        assert np.array_equal(d_out[r].host(), want[r]) and d_out[r].guards_intact()
    assert np.array_equal(extra_dst.host(), extra_src.host()) and extra_dst.guards_intact()


@pytest.mark.parametrize("n,nb", [(9, 8 * MiB), (64, 1 * MiB), (65, 1 * MiB), (200, 512 * KiB), (70, 100 * KiB),
                                  (100, 4 * MiB)])
def test_long_lists_of_equal_large_copies(ref, n, nb):
    """Lists of equal, aligned, large copies, which travel in the kernel arguments: up to 64 of them as they are, longer
    lists as offsets (the lists that do need a table: test_equal_copies_from_a_staged_table); every byte of the arena is
    compared."""
    run_batch(ref, n, nb, 2 * n * nb + 64 * MiB, seed=n, align=4096)


def test_alltoall_uniform_2MiB_chunks_every_chunk(ref):
    run_alltoall(ref, inputs.uniform_chunks(8, 2 * MiB), seed=3, kind="fp16")


# ------------------------------------------- KV-cache fetch / save (Sec. V-C)

@pytest.mark.parametrize("block_bytes", [16 * KiB, 160 * KiB, 1 * MiB + 4096])
def test_kv_fetch_from_pinned_host_memory_and_save_back(ref, block_bytes):
    """256 dispersed blocks per request, host-pinned pool -> device pool in one batch (fetch), then
    a different set device -> host (save).  The checker sees the same two pools as host arrays."""
    import torch
    n, host_blocks, dev_blocks = 256, 300, 280
    rng = np.random.default_rng(block_bytes)
    host_pool = rng.integers(0, 256, host_blocks * block_bytes, dtype=np.uint8)
    dev_pool = rng.integers(0, 256, dev_blocks * block_bytes, dtype=np.uint8)
    pinned = torch.empty(host_pool.size, dtype=torch.uint8, pin_memory=True)
    pinned.copy_(torch.from_numpy(host_pool))
    d = DevBuf(dev_pool.size, fill=dev_pool)
    hp = pinned.data_ptr()

    pairs = inputs.kv_fetch_blocks(n, host_blocks, dev_blocks, seed=1)
    want_h, want_d = ref.batch_copy([host_pool.copy(), dev_pool.copy()],
                                    [(0, int(s) * block_bytes, 1, int(t) * block_bytes, block_bytes) for s, t in pairs])
    dl.dl_batch_copy([(hp + int(s) * block_bytes, d.ptr(int(t) * block_bytes), block_bytes) for s, t in pairs], stream())
    sync()
    assert np.array_equal(d.host(), want_d) and d.guards_intact()
    assert np.array_equal(pinned.numpy(), want_h)

    pairs = inputs.kv_fetch_blocks(n, host_blocks, dev_blocks, seed=2)
    want_h, want_d = ref.batch_copy([want_h, want_d],
                                    [(1, int(t) * block_bytes, 0, int(s) * block_bytes, block_bytes) for s, t in pairs])
    dl.dl_batch_copy([(d.ptr(int(t) * block_bytes), hp + int(s) * block_bytes, block_bytes) for s, t in pairs], stream())
    sync()
    assert np.array_equal(pinned.numpy(), want_h)
    assert np.array_equal(d.host(), want_d) and d.guards_intact()


# ------------------------------------------------- swap / in-place all-to-all

def run_swaps(ref, n, nb, arena_bytes, seed, align=256):
    arena, descs = inputs.swap_batch(n, nb, arena_bytes, seed, align)
    want = ref.batch_swap([arena.copy()], [(0, a, 0, b, m) for a, b, m in descs])[0]
    d = DevBuf(arena_bytes, fill=arena)
    dl.dl_batch_swap([(d.ptr(int(a)), d.ptr(int(b)), int(m)) for a, b, m in descs], stream())
    sync()
    assert np.array_equal(d.host(), want)
    assert d.guards_intact()


@pytest.mark.parametrize("n,nb,arena,align", [(1, 100, 4096, 1), (4, 16 * KiB, 1 * MiB, 256), (7, 5000, 256 * KiB, 16),
                                              (8, 1 * MiB + 48, 32 * MiB, 256), (40, 70001, 16 * MiB, 1),
                                              (40, 4096, 4 * MiB, 4), (300, 3000, 8 * MiB, 8)])
def test_batch_swap_shapes(ref, n, nb, arena, align):
    """Row path (aligned, short list), general path (ragged, modulo 4, modulo 1), long lists (table kernel)."""
    run_swaps(ref, n, nb, arena, seed=n + nb, align=align)


def run_alltoall_inplace(ref, W, c, seed, kind="u8"):
    bufs = inputs.alltoall_inputs(inputs.uniform_chunks(W, c), seed=seed, kind=kind)
    want = ref.alltoall_inplace(bufs, c)
    d = [DevBuf(W * c, fill=bufs[i]) for i in range(W)]
    dl.dl_alltoall_inplace([b.ptr() for b in d], c, stream())
    sync()
    for i in range(W):
        assert np.array_equal(d[i].host(), want[i]), f"rank {i} differs (W={W}, c={c})"
        assert d[i].guards_intact()
    return d, bufs


@pytest.mark.parametrize("c", [1 * KiB, 64 * KiB, 4 * MiB])
def test_alltoall_inplace_uniform_fp16(ref, c):
    run_alltoall_inplace(ref, 8, c, seed=c, kind="fp16")


@pytest.mark.parametrize("W,c", [(1, 1000), (2, 17), (3, 4097), (5, 16), (8, 1), (8, 100001), (13, 5000)])
def test_alltoall_inplace_ranks_and_ragged_chunks(ref, W, c):
    run_alltoall_inplace(ref, W, c, seed=W * 1000 + c)


def test_alltoall_inplace_twice_is_identity_and_matches_out_of_place(ref):
    W, c = 8, 48 * KiB
    d, bufs = run_alltoall_inplace(ref, W, c, seed=77, kind="bf16")
    # the out-of-place operation on the same inputs gives the same buffers
    d_in = [DevBuf(W * c, fill=bufs[i]) for i in range(W)]
    d_out = [DevBuf(W * c) for _ in range(W)]
    dl.dl_alltoall([b.ptr() for b in d_in], [b.ptr() for b in d_out], inputs.uniform_chunks(W, c), stream())
    dl.dl_alltoall_inplace([b.ptr() for b in d], c, stream())
    sync()
    for i in range(W):
        assert np.array_equal(d_out[i].host(), ref.alltoall_inplace(bufs, c)[i])
        assert np.array_equal(d[i].host(), bufs[i])


def test_swap_validation_rejects_overlap_and_enqueues_nothing():
    d = DevBuf(4096)
    before = d.host().copy()
    dl.dl_set_validate(True)
    try:
        with pytest.raises(dl.DlError) as e:
            dl.dl_batch_swap([(d.ptr(0), d.ptr(1000), 500), (d.ptr(1400), d.ptr(2000), 500)], stream())
        assert e.value.status == dl.DL_ERR_OVERLAP
        with pytest.raises(dl.DlError) as e:
            dl.dl_batch_swap([(d.ptr(0), d.ptr(100), 500)], stream())
        assert e.value.status == dl.DL_ERR_OVERLAP
    finally:
        dl.dl_set_validate(VALIDATE_ALL)
    sync()
    assert np.array_equal(d.host(), before)


@pytest.mark.parametrize("shift", [0, 4, 1])
def test_items_longer_than_4GiB(ref, shift):
    """Byte offsets inside one item pass 2^32: a single copy and a 1 -> 2 broadcast of 4 GiB + 4112 bytes, with
    the destinations aligned like the source (16-byte path), 4 bytes off (4-byte path) and 1 byte off (byte
    path).  Too long for the CPU checker within a test's time: the device compares every byte with the source
    (a copy has no other correct result), and the checker runs on windows around the start, 2^31, 2^32 and the end."""
    import torch
    n = (4 << 30) + 4112
    src = DevBuf(n)
    src.view().random_(0, 256)
    d1, d2 = DevBuf(n, shift=shift), DevBuf(n, shift=shift)
    dl.dl_batch_copy([(src.ptr(), d1.ptr(), n)], stream())
    sync()
    assert torch.equal(d1.view(), src.view()) and d1.guards_intact()
    d1.view().zero_()
    dl.dl_broadcast(src.ptr(), [d1.ptr(), d2.ptr()], n, stream())
    sync()
    assert torch.equal(d1.view(), src.view()) and torch.equal(d2.view(), src.view())
    assert d1.guards_intact() and d2.guards_intact() and src.guards_intact()
    for lo in (0, (1 << 31) - 2048, (1 << 32) - 2048, n - 4096):
        win = src.view()[lo:lo + 4096].cpu().numpy()
        want = ref.broadcast(win, 2)
        assert np.array_equal(d1.view()[lo:lo + 4096].cpu().numpy(), want[0])
        assert np.array_equal(d2.view()[lo:lo + 4096].cpu().numpy(), want[1])


def test_swap_and_allgather_beyond_4GiB(ref):
    """A swap of two ranges of 4 GiB + 48 bytes, and an all-gather whose receive offsets j * B pass 2^32
    (W = 3, B = 2 GiB + 16); compared on the device with what the definitions give."""
    import torch
    n = (4 << 30) + 48
    a, b = DevBuf(n), DevBuf(n)
    a.view().random_(0, 256)
    b.view().random_(0, 256)
    a0, b0 = a.view().clone(), b.view().clone()
    dl.dl_batch_swap([(a.ptr(), b.ptr(), n)], stream())
    sync()
    assert torch.equal(a.view(), b0) and torch.equal(b.view(), a0) and a.guards_intact() and b.guards_intact()
    del a, b, a0, b0
    W, B = 3, (2 << 30) + 16
    d_in = [DevBuf(B) for _ in range(W)]
    for t in d_in:
        t.view().random_(0, 256)
    d_out = [DevBuf(W * B) for _ in range(W)]
    dl.dl_allgather([t.ptr() for t in d_in], [t.ptr() for t in d_out], B, stream())
    sync()
    for r in range(W):
        for j in range(W):
            assert torch.equal(d_out[r].view()[j * B:(j + 1) * B], d_in[j].view()), (r, j)
        assert d_out[r].guards_intact()
    lo = B - 2048                                   # a window across the first block boundary, against the checker
    want = ref.allgather([t.view()[lo:].cpu().numpy() for t in d_in])
    for r in range(W):
        for j in range(W):
            got = d_out[r].view()[j * B + lo:(j + 1) * B].cpu().numpy()
            assert np.array_equal(got, want[r][j * 2048:(j + 1) * 2048])


def test_short_one_shot_requests_replay_from_a_graph(ref):
    """A one-shot request whose list fits the kernel arguments is exactly one kernel launch on the caller's
    stream (no allocation, no copy, no event), so a caller can capture it in a HIP graph.  Three requests are
    captured once and replayed with new source bytes each time; every replay is compared with the checker, with
    eager work and synchronisations in between."""
    import torch
    W, B, c, n = 8, 16 * KiB, 4 * KiB, 300 * KiB + 48
    rng = np.random.default_rng(11)
    ag_in = [DevBuf(B) for _ in range(W)]
    ag_out = [DevBuf(W * B) for _ in range(W)]
    C = inputs.uniform_chunks(W, c)
    aa_in = [DevBuf(W * c) for _ in range(W)]
    aa_out = [DevBuf(W * c) for _ in range(W)]
    bc_src = DevBuf(n)
    bc_dst = [DevBuf(n) for _ in range(5)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        cap = torch.cuda.current_stream()
        dl.dl_allgather([b.ptr() for b in ag_in], [b.ptr() for b in ag_out], B, cap)
        dl.dl_alltoall([b.ptr() for b in aa_in], [b.ptr() for b in aa_out], C, cap)
        dl.dl_broadcast(bc_src.ptr(), [b.ptr() for b in bc_dst], n, cap)
    for replay in range(4):
        ins = [rng.integers(0, 256, B, dtype=np.uint8) for _ in range(W)]
        aas = [rng.integers(0, 256, W * c, dtype=np.uint8) for _ in range(W)]
        src = rng.integers(0, 256, n, dtype=np.uint8)
        for b, a in zip(ag_in + aa_in + [bc_src], ins + aas + [src]):
            b.view().copy_(torch.from_numpy(a))
        for b in ag_out + aa_out + bc_dst:
            b.view().zero_()
        sync()
        g.replay()
        torch.cuda.synchronize()
        for r, w in zip(ag_out, ref.allgather(ins)):
            assert np.array_equal(r.host(), w) and r.guards_intact(), f"all-gather, replay {replay}"
        for r, w in zip(aa_out, ref.alltoall(aas, C)):
            assert np.array_equal(r.host(), w) and r.guards_intact(), f"all-to-all, replay {replay}"
        for r in bc_dst:
            assert np.array_equal(r.host(), src) and r.guards_intact(), f"broadcast, replay {replay}"


def test_empty_requests_are_no_ops():
    d = DevBuf(1024)
    dl.dl_batch_copy([], stream())
    dl.dl_batch_copy([(d.ptr(), d.ptr(512), 0), (d.ptr(5), d.ptr(5), 100)], stream())
    dl.dl_allgather([d.ptr()], [d.ptr(512)], 0, stream())
    dl.dl_broadcast(d.ptr(), [d.ptr(512)], 0, stream())
    dl.dl_alltoall([d.ptr(), d.ptr(8)], [d.ptr(512), d.ptr(600)], np.zeros((2, 2), dtype=np.uint64), stream())
    dl.dl_batch_swap([], stream())
    dl.dl_batch_swap([(d.ptr(), d.ptr(512), 0), (d.ptr(7), d.ptr(7), 100)], stream())
    dl.dl_alltoall_inplace([d.ptr(), d.ptr(512)], 0, stream())
    sync()
    assert (d.host() == 0xA5).all()


def test_validation_rejects_hazards_and_enqueues_nothing():
    d = DevBuf(4096)
    before = d.host().copy()
    dl.dl_set_validate(True)
    try:
        with pytest.raises(dl.DlError) as e:
            dl.dl_batch_copy([(d.ptr(0), d.ptr(1000), 500), (d.ptr(2000), d.ptr(1400), 500)], stream())
        assert e.value.status == dl.DL_ERR_OVERLAP
        with pytest.raises(dl.DlError) as e:
            dl.dl_broadcast(d.ptr(0), [d.ptr(1000), d.ptr(50)], 100, stream())
        assert e.value.status == dl.DL_ERR_OVERLAP
        dl.dl_batch_copy([(d.ptr(0), d.ptr(1000), 500), (d.ptr(100), d.ptr(1500), 500)], stream())
    finally:
        dl.dl_set_validate(VALIDATE_ALL)
    sync()
    after = d.host()
    assert np.array_equal(after[:1000], before[:1000]) and np.array_equal(after[2000:], before[2000:])
    assert np.array_equal(after[1000:1500], before[0:500]) and np.array_equal(after[1500:2000], before[100:600])


# ----------------------------------- failure reports from the device; table memory after a stream has gone

def lib_error_pending():
    """Whether a loss has been reported, without clearing the report: an empty request is refused while it is."""
    try:
        dl.dl_batch_copy_static([(1 << 20, 2 << 20, 0)], stream())   # moves nothing, enqueues nothing
    except dl.DlError as e:
        assert e.status == dl.DL_ERR_LOST
        return True
    return False


def _lose_next_table():
    """Arm the test hook, or skip where no table goes through the BAR."""
    try:
        dl.dl_debug_lose_next_table(3)
    except dl.DlError as e:
        if e.status == dl.DL_ERR_STATE:
            pytest.skip("no table is written through the BAR in this configuration")
        raise


@pytest.mark.parametrize("kind", ["table", "rows_table", "token_dispatch"])
def test_a_table_that_never_completes_is_reported_and_nothing_is_copied(ref, kind):
    """The kernel of a long list is told (by the test hook) a stamp that its table's slot will never hold, and
    three looks: every workgroup gives up its bounded wait and leaves.  The call has returned DL_OK long before;
    the loss shows in dl_last_device_error(), every operation refuses until it has been read, no destination
    byte has changed, and the same request issued again gives the oracle's result."""
    assert dl.dl_last_device_error() == dl.DL_OK
    W = 8
    if kind == "token_dispatch":
        counts, row = [300] * W, 512     # 2400 tokens: more than the kernel arguments hold
        ins = inputs.token_rows(W, counts, row, seed=5, kind="u8")
        dest = inputs.moe_token_destinations(W, counts, seed=6, n_experts=256, top_k=8)
        want = ref.token_dispatch(ins, row, dest)
        d_in = [DevBuf(a.size, fill=a) for a in ins]
        outs = [DevBuf(w.size, fill=np.full(w.size, 0x3C, dtype=np.uint8)) for w in want]
        before = [np.full(w.size, 0x3C, dtype=np.uint8) for w in want]

        def issue():
            dl.dl_token_dispatch([b.ptr() for b in d_in], [b.ptr() for b in outs], counts, row, dest, stream())
    else:
        # equal copies: more than fit the kernel arguments as offsets, too small for several launches
        arena, descs = inputs.b2b_batch(500, 16 * KiB, 64 * MiB, seed=500) if kind == "rows_table" else \
            inputs.mixed_batch(300, 5000, 8 * MiB, seed=300)
        want = [ref.batch_copy([arena.copy()], [(0, s, 0, d, m) for s, d, m in descs])[0]]
        outs = [DevBuf(arena.size, fill=arena)]
        before = [arena]

        def issue():
            d = outs[0]
            dl.dl_batch_copy([(d.ptr(int(s)), d.ptr(int(t)), int(m)) for s, t, m in descs], stream())

    _lose_next_table()
    try:
        issue()
    finally:
        dl.dl_debug_lose_next_table(0)    # taken back if no table took it
    sync()
    if FORCED and not lib_error_pending():
        pytest.skip("with these forced settings the request's table does not go through the BAR")
    with pytest.raises(dl.DlError) as refused:
        issue()
    assert refused.value.status == dl.DL_ERR_LOST
    assert dl.dl_last_device_error() == dl.DL_ERR_LOST
    assert dl.dl_last_device_error() == dl.DL_OK
    for d, b in zip(outs, before):
        assert np.array_equal(d.host(), b) and d.guards_intact(), "a request whose table was lost changed a byte"
    issue()
    sync()
    assert dl.dl_last_device_error() == dl.DL_OK
    for d, w in zip(outs, want):
        assert np.array_equal(d.host(), w) and d.guards_intact()


def test_requests_without_a_table_do_not_heed_the_lost_table_hook(ref):
    """Equal copies at offsets and a token dispatch of 640 tokens travel in the kernel arguments: with the hook armed
    they run as ever, and the next table, of unequal copies, is the one that is lost."""
    W, counts, row = 8, [80] * 8, 512
    ins = inputs.token_rows(W, counts, row, seed=5, kind="u8")
    dest = inputs.moe_token_destinations(W, counts, seed=6, n_experts=256, top_k=8)
    want = ref.token_dispatch(ins, row, dest)
    d_in = [DevBuf(a.size, fill=a) for a in ins]
    outs = [DevBuf(w.size) for w in want]
    arena, descs = inputs.b2b_batch(200, 16 * KiB, 32 * MiB, seed=200)
    d = DevBuf(arena.size, fill=arena)
    arena2, descs2 = inputs.mixed_batch(300, 5000, 8 * MiB, seed=301)
    d2 = DevBuf(arena2.size, fill=arena2)

    def copy(buf, ds):
        dl.dl_batch_copy([(buf.ptr(int(s)), buf.ptr(int(t)), int(m)) for s, t, m in ds], stream())

    assert dl.dl_last_device_error() == dl.DL_OK
    _lose_next_table()
    try:
        dl.dl_token_dispatch([b.ptr() for b in d_in], [b.ptr() for b in outs], counts, row, dest, stream())
        for request in (None, descs):
            if request is not None:
                copy(d, request)
            sync()
            if FORCED and lib_error_pending():
                pytest.skip("with these forced settings one of the requests has a table")
        assert dl.dl_last_device_error() == dl.DL_OK
        copy(d2, descs2)
        sync()
        if FORCED and not lib_error_pending():
            pytest.skip("with these forced settings the list's table does not go through the BAR")
    finally:
        dl.dl_debug_lose_next_table(0)
        lost = dl.dl_last_device_error()
    assert lost == dl.DL_ERR_LOST
    for b, w in zip(outs, want):
        assert np.array_equal(b.host(), w) and b.guards_intact()
    assert np.array_equal(d.host(), ref.batch_copy([arena.copy()], [(0, s, 0, t, m) for s, t, m in descs])[0]) and d.guards_intact()
    assert np.array_equal(d2.host(), arena2)


def _hip_runtime():
    """The HIP runtime this process has loaded already (the one that owns every stream here)."""
    import ctypes
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert paths, "no HIP runtime loaded"
    return ctypes.CDLL(sorted(paths)[0])


@pytest.mark.parametrize("push", [1, 0])
def test_table_memory_is_reused_after_the_callers_stream_is_gone(ref, cfg, push):
    """A long-list request on a stream of the caller's, which the caller destroys once it has synchronised; then
    enough long-list requests on the default stream that every table slot is used again.  The library must not
    touch the dead stream (its event was recorded while the stream was alive).  The copies of a request have unequal
    lengths: equal ones travel in the kernel arguments and use no table."""
    import ctypes
    import torch
    cfg(table_push=push)
    hip = _hip_runtime()
    hip.hipStreamCreate.argtypes = [ctypes.POINTER(ctypes.c_void_p)]
    hip.hipStreamSynchronize.argtypes = [ctypes.c_void_p]
    hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    rng = np.random.default_rng(5)
    cases = []
    for r in range(71):
        n = int(rng.integers(80, 300))
        arena, descs = inputs.mixed_batch(n, int(rng.choice([512, 3000, 16 * KiB])), 16 * MiB, seed=100 + r)
        lengths = descs[:, 2][descs[:, 2] > 0]
        assert len(lengths) > 64 and len(set(lengths.tolist())) > 1, "a request that needs no table"
        cases.append((arena, DevBuf(arena.size, fill=arena), descs))
    torch.cuda.synchronize()

    def issue(case, st):
        _, d, descs = case
        dl.dl_batch_copy([(d.ptr(int(s)), d.ptr(int(t)), int(m)) for s, t, m in descs], st)

    own = ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(own)) == 0
    issue(cases[0], own.value)
    assert hip.hipStreamSynchronize(own) == 0
    assert hip.hipStreamDestroy(own) == 0
    for case in cases[1:]:
        issue(case, stream())
    sync()
    for r, (arena, d, descs) in enumerate(cases):
        want = ref.batch_copy([arena.copy()], [(0, s, 0, t, m) for s, t, m in descs])[0]
        assert np.array_equal(d.host(), want) and d.guards_intact(), f"request {r}"


def test_tunables_from_the_environment(ref):
    """DL_CONFIG is applied by dl_init on top of the defaults (a process of its own: the library of this process
    is initialised already); a value that does not parse makes dl_init fail."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    child = (
        "import sys, numpy as np, torch\n"
        f"sys.path.insert(0, {root!r})\n"
        "import paper_2511_06605_amd as dl\n"
        "from paper_2511_06605_amd import inputs\n"
        "from oracle import ref\n"
        "torch.cuda.set_device(0)\n"
        "try:\n"
        "    dl.dl_init(0)\n"
        "except dl.DlError as e:\n"
        "    print('init refused', e.status); sys.exit(0)\n"
        "c = dl.dl_get_config()\n"
        "print('config', c.fan_split, c.table_push, c.tile_bytes, c.infer_broadcast)\n"
        "ins = inputs.allgather_inputs(8, 50000, seed=1)\n"
        "d_in = [torch.from_numpy(a).cuda() for a in ins]\n"
        "d_out = [torch.zeros(8 * 50000, dtype=torch.uint8, device='cuda') for _ in range(8)]\n"
        "dl.dl_allgather(d_in, d_out, 50000, torch.cuda.current_stream()); torch.cuda.synchronize()\n"
        "assert all(np.array_equal(g.cpu().numpy(), w) for g, w in zip(d_out, ref.allgather(ins)))\n"
        "dl.dl_shutdown(); print('result ok')\n")

    def run(text):
        env = dict(os.environ, DL_CONFIG=text)
        return subprocess.run([sys.executable, "-c", child], capture_output=True, text=True, env=env, timeout=120)

    r = run("fan_split=2,table_push=0")
    assert "config 2 0 0 1" in r.stdout and "result ok" in r.stdout, r.stdout + r.stderr
    r = run("fan_split=3")
    assert f"init refused {dl.DL_ERR_INVALID}" in r.stdout, r.stdout + r.stderr
