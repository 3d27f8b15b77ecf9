"""The marshalling module's calls (csrc/dl_marshal.c) made with ctypes objects, for a Python that has no extension built
for it (no headers where the library was built, or another Python than the one that built it).  Same arguments, same
results; a call takes longer (all-gather of 2 KiB over eight ranks 9.5 us against 7.2, 256 copies 66.5 against 10.5).
Every function holds its buffers until the library has returned.
"""

from __future__ import annotations

import ctypes

from . import binding as b

NAMES = ()


def bind(addresses) -> None:
    """Nothing to bind: the entry points are looked up in the loaded library at each call."""
    list(addresses)


def _pair(ins, outs):
    ins, outs = list(ins), list(outs)
    if len(ins) != len(outs):
        raise ValueError("need as many receive buffers as send buffers")
    return ins, outs


def allgather(ins, outs, bytes_per_rank, stream):
    ins, outs = _pair(ins, outs)
    return b.lib().dl_allgather(b._ptr_array(ins), b._ptr_array(outs), len(ins), int(bytes_per_rank), b._stream(stream))


def alltoall(ins, outs, chunk_bytes, stream):
    ins, outs = _pair(ins, outs)
    W = len(ins)
    return b.lib().dl_alltoall(b._ptr_array(ins), b._ptr_array(outs), W, b._chunk_array(chunk_bytes, W), b._stream(stream))


def alltoall_inplace(bufs, chunk_bytes, stream):
    bufs = list(bufs)
    return b.lib().dl_alltoall_inplace(b._ptr_array(bufs), len(bufs), int(chunk_bytes), b._stream(stream))


def broadcast(src, dsts, nbytes, stream):
    dsts = list(dsts)
    return b.lib().dl_broadcast(b._addr(src), b._ptr_array(dsts), len(dsts), int(nbytes), b._stream(stream))


def batch_copy(descs, stream):
    descs = list(descs)
    return b.lib().dl_batch_copy(b._desc_array(descs), len(descs), b._stream(stream))


def batch_copy_static(descs, stream):
    descs = list(descs)
    return b.lib().dl_batch_copy_static(b._desc_array(descs), len(descs), b._stream(stream))


def batch_swap(descs, stream):
    descs = list(descs)
    return b.lib().dl_batch_swap(b._swap_array(descs), len(descs), b._stream(stream))


def token_dispatch(ins, outs, tokens, row_bytes, dest, stream):
    ins, outs = list(ins), list(outs)
    i, o, W, tok, d = b._dispatch_args(ins, outs, tokens, dest)
    return b.lib().dl_token_dispatch(i, o, W, tok, int(row_bytes), d, b._stream(stream))


def token_dispatch_device(ins, outs, tokens, row_bytes, dest_device, stream):
    ins, outs = list(ins), list(outs)
    W = len(ins)
    if len(outs) != W or len(tokens) != W:
        raise ValueError("need W send buffers, W receive buffers and W token counts")
    tok = (ctypes.c_uint32 * W)(*[int(t) for t in tokens])
    return b.lib().dl_token_dispatch_device(b._ptr_array(ins), b._ptr_array(outs), W, tok, int(row_bytes), b._addr(dest_device),
                                            b._stream(stream))


def set_mode(mode):
    return b.lib().dl_set_mode(mode)


def last_ticket():
    return int(b.lib().dl_last_ticket())


def trigger(ticket):
    return b.lib().dl_trigger(ticket)


def wait(ticket, timeout_ns):
    return b.lib().dl_wait(ticket, timeout_ns)
