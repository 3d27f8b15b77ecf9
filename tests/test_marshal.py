"""The marshalling module against the ctypes helpers: what the library's entry points are handed, recorded by stubs
in their place (no GPU, no library call)."""

import ctypes
import os
import re
import shutil
import subprocess
import sysconfig

import numpy as np
import pytest

from paper_2511_06605_amd import binding, build

vp, sz, u64, u32 = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_uint64, ctypes.c_uint32
PP = ctypes.POINTER(vp)


class Tensor:
    def __init__(self, p):
        self.p = p

    def data_ptr(self):
        return self.p

    def __index__(self):     # a one-element tensor has a value as well: not what is wanted
        return 7


class Stream:
    cuda_stream = 0xABC0


stubs = {}  # the entry points that `calls` put in place, by name


@pytest.fixture()
def calls():
    """Binds the module to stubs that note their arguments as Python values; the real entry points afterwards."""
    L, m = binding.lib(), binding._native()
    seen = []

    def words(p, n):
        return [p[i] or 0 for i in range(n)]

    def triples(p, n):
        q = ctypes.cast(p, ctypes.POINTER(u64)) if n else None
        return [tuple(q[3 * i:3 * i + 3]) for i in range(n)]

    def note(name, f):
        def g(*a):
            seen.append((name,) + f(*a))
            return -5
        return g

    def dispatch(i, o, W, t, row, d, s):
        n = sum(t[:W])
        return words(i, W), words(o, W), list(t[:W]), row, d or 0, s or 0, (bytes((ctypes.c_uint8 * (n * W)).from_address(d)) if d and d < 1 << 60 else None)

    kinds = {
        "dl_allgather": ([PP, PP, ctypes.c_int, sz, vp], lambda i, o, W, b, s: (words(i, W), words(o, W), b, s or 0)),
        "dl_alltoall": ([PP, PP, ctypes.c_int, ctypes.POINTER(sz), vp], lambda i, o, W, c, s: (words(i, W), words(o, W), list(c[:W * W]), s or 0)),
        "dl_alltoall_inplace": ([PP, ctypes.c_int, sz, vp], lambda b, W, c, s: (words(b, W), c, s or 0)),
        "dl_broadcast": ([vp, PP, ctypes.c_int, sz, vp], lambda a, d, k, b, s: (a or 0, words(d, k), b, s or 0)),
        "dl_batch_copy": ([vp, sz, vp], lambda p, n, s: (triples(p, n), s or 0)),
        "dl_batch_copy_static": ([vp, sz, vp], lambda p, n, s: (triples(p, n), s or 0)),
        "dl_batch_swap": ([vp, sz, vp], lambda p, n, s: (triples(p, n), s or 0)),
        "dl_token_dispatch": ([PP, PP, ctypes.c_int, ctypes.POINTER(u32), sz, vp, vp], dispatch),
        "dl_token_dispatch_device": ([PP, PP, ctypes.c_int, ctypes.POINTER(u32), sz, vp, vp], dispatch),
        "dl_set_mode": ([ctypes.c_int], lambda v: (v,)),
        "dl_trigger": ([u64], lambda v: (v,)),
        "dl_wait": ([u64, u64], lambda t, ns: (t, ns)),
    }
    keep = []
    for name in m.NAMES:
        if name == "dl_last_ticket":
            keep.append(ctypes.CFUNCTYPE(u64)(lambda: 2 ** 63 + 1))
        else:
            keep.append(ctypes.CFUNCTYPE(ctypes.c_int, *kinds[name][0])(note(name, kinds[name][1])))
    m.bind([ctypes.cast(f, vp).value for f in keep])
    stubs.clear()
    stubs.update(zip(m.NAMES, keep))
    yield m, seen
    m.bind([ctypes.cast(getattr(L, n), vp).value for n in m.NAMES])


A = [0x10, Tensor(0x2000000000), None, np.uint64(0x7FFFFFFFFFFF)]
A_WORDS = [0x10, 0x2000000000, 0, 0x7FFFFFFFFFFF]


@pytest.mark.parametrize("stream,handle", [(None, 0), (0, 0), (0x77, 0x77), (Stream(), 0xABC0)])
def test_pointer_lists_and_streams(calls, stream, handle):
    m, seen = calls
    B = [Tensor(2 ** 63), 1, 2, 3]
    assert m.allgather(A, tuple(B), np.int64(4096), stream) == -5
    assert m.allgather((x for x in A), iter(B), 5.0, stream) == -5
    assert m.alltoall_inplace(A, 2 ** 33, stream) == -5
    assert m.broadcast(Tensor(0x99), A, 1, stream) == -5
    assert m.allgather(range(1, 70), range(1, 70), 1, stream) == -5            # more than fits the stack
    assert m.allgather([], [], 1, stream) == -5
    assert seen == [("dl_allgather", A_WORDS, [2 ** 63, 1, 2, 3], 4096, handle), ("dl_allgather", A_WORDS, [2 ** 63, 1, 2, 3], 5, handle),
                    ("dl_alltoall_inplace", A_WORDS, 2 ** 33, handle), ("dl_broadcast", 0x99, A_WORDS, 1, handle),
                    ("dl_allgather", list(range(1, 70)), list(range(1, 70)), 1, handle), ("dl_allgather", [], [], 1, handle)]
    assert words_of(binding._ptr_array(A)) == A_WORDS


def words_of(arr):
    return [v or 0 for v in arr]


@pytest.mark.parametrize("chunks", [[[1, 2], [3, 2 ** 40]], np.array([[1, 2], [3, 2 ** 40]], dtype=np.uint64), [1, 2, 3, 2 ** 40],
                                    np.array([1, 2, 3, 2 ** 40]), [[1, 2], 3, 2 ** 40], [(1.0, 2), np.array([3, 2 ** 40])]])
def test_chunk_matrices(calls, chunks):
    m, seen = calls
    assert m.alltoall([8, 9], [10, 11], chunks, 3) == -5
    assert seen == [("dl_alltoall", [8, 9], [10, 11], [1, 2, 3, 2 ** 40], 3)]
    assert list(binding._chunk_array(chunks, 2)) == [1, 2, 3, 2 ** 40]


@pytest.mark.parametrize("call,name", [("batch_copy", "dl_batch_copy"), ("batch_copy_static", "dl_batch_copy_static"), ("batch_swap", "dl_batch_swap")])
def test_triples(calls, call, name):
    m, seen = calls
    f = getattr(m, call)
    descs = [(0x10, Tensor(0x20), 3), [Tensor(5), None, np.int32(9)], np.array([1, 2, 3], dtype=np.uint64)]
    assert f(descs, None) == -5 and f(iter(descs), Stream()) == -5 and f([], 1) == -5
    got = [(0x10, 0x20, 3), (5, 0, 9), (1, 2, 3)]
    assert seen == [(name, got, 0), (name, got, 0xABC0), (name, [], 1)]
    for bad in ([(1, 2)], [(1, 2, 3, 4)], [()]):
        with pytest.raises(ValueError):
            f(bad, None)
    for bad in ([(1, 2, "x")], [("x", 2, 3)], [(1, 2, None)], [5], 5):
        with pytest.raises((TypeError, ValueError)):
            f(bad, None)
    assert len(seen) == 3


# integers read where they lie: none to three digits of 30 bits, signs, what is no exact int, not a triple or no tuple, at the
# front of a list and behind others
@pytest.mark.parametrize("call,name", [("batch_copy", "dl_batch_copy"), ("batch_swap", "dl_batch_swap")])
def test_triples_of_integers(calls, call, name):
    m, seen = calls
    edges = [0, 1, 2 ** 30 - 1, 2 ** 30, 2 ** 47 + 5, 2 ** 60 - 1, 2 ** 60, 2 ** 63, 2 ** 64 - 1, 2 ** 70 + 3, -1, -2 ** 31, True]
    plain = [(v, 2 ** 40 + v, 7) for v in edges if v is not True]
    odd = [(True, 1, 2), [1, 2, 3], (Tensor(0x99), 4, 5), (np.int64(6), 7, np.uint8(8)), (None, 1, 2), range(3)]
    mask = 2 ** 64 - 1

    def words(t):
        return tuple((binding._addr(v) or 0) & mask if i < 2 else int(v) & mask for i, v in enumerate(t))

    for descs in [plain, plain[:5], *([o] + plain[:3] for o in odd), *(plain[:3] + [o] + plain[3:] for o in odd)]:
        for form in (list, tuple, iter):
            seen.clear()
            assert getattr(m, call)(form(descs), None) == -5
            assert seen == [(name, [words(t) for t in descs], 0)]
    for bad in (plain[:2] + [(1, 2)], [(1, 2, 3, 4)], [(1, 2, 3), 5], [(1, 2, "x")], [("x", 1, 2)]):
        seen.clear()
        with pytest.raises((TypeError, ValueError)):
            getattr(m, call)(bad, None)
        assert not seen


def test_dispatch_masks(calls):
    m, seen = calls
    mask = np.arange(6, dtype=np.uint8).reshape(3, 2)
    assert m.token_dispatch([1, 2], [3, 4], [2, np.int32(1)], 16, mask, 9) == -5
    assert m.token_dispatch([1, 2], [3, 4], [2, 1], 16, mask != 0, None) == -5
    assert m.token_dispatch([1, 2], [3, 4], [2, 1], 16, bytes(6), None) == -5
    assert [c[1:5] for c in seen] == [([1, 2], [3, 4], [2, 1], 16)] * 3
    assert [c[7] for c in seen] == [bytes(range(6)), b"\0" + b"\1" * 5, bytes(6)]
    for other in (mask.astype(np.int32), mask.T, mask.tolist(), np.asfortranarray(mask), mask[::-1]):
        assert m.token_dispatch([1, 2], [3, 4], [2, 1], 16, other, None) is NotImplemented
    with pytest.raises(ValueError):
        m.token_dispatch([1, 2], [3, 4], [2, 2], 16, mask, None)
    with pytest.raises(ValueError):
        m.token_dispatch([1, 2], [3, 4], [3], 16, mask, None)
    assert m.token_dispatch_device([1, 2], [3, 4], [2, 1], 16, Tensor(2 ** 62), None) == -5
    assert seen[-1][:6] == ("dl_token_dispatch_device", [1, 2], [3, 4], [2, 1], 16, 2 ** 62)
    assert len(seen) == 4


def test_small_calls_and_errors(calls):
    m, seen = calls
    assert m.set_mode(-1) == -5 and m.trigger(2 ** 64 - 1) == -5 and m.wait(np.uint64(3), 5_000_000_000) == -5
    assert m.last_ticket() == 2 ** 63 + 1
    assert seen == [("dl_set_mode", -1), ("dl_trigger", 2 ** 64 - 1), ("dl_wait", 3, 5_000_000_000)]

    class Broken:
        def data_ptr(self):
            raise RuntimeError("no storage")

    with pytest.raises(RuntimeError):
        m.allgather([Broken()], [1], 1, None)
    with pytest.raises(ValueError):
        m.allgather([1], [1, 2], 1, None)
    with pytest.raises(ValueError):
        m.alltoall([1, 2], [1, 2], [[1, 2], [3]], None)
    with pytest.raises(ValueError):
        m.alltoall([1, 2], [1, 2], [[1, 2], [3, 4, 5]], None)
    for args in ((), (1,), ([1], [1], 1), ([1], [1], 1, None, None), ([1], [1], "x", None), ([1], [1], 1, "x"), (3, [1], 1, None)):
        with pytest.raises((TypeError, ValueError)):
            m.allgather(*args)
    assert len(seen) == 3


class Block:
    """A buffer from an allocator that hands the lowest free address out, as a caching allocator does."""
    live = set()

    def __init__(self):
        self.p = next(a for a in range(0x1000, 1 << 20, 0x1000) if a not in Block.live)
        Block.live.add(self.p)

    def __del__(self):
        Block.live.discard(self.p)

    def data_ptr(self):
        return self.p


def fresh(n):
    return (Block() for _ in range(n))


@pytest.mark.parametrize("call", [
    lambda m: m.allgather(fresh(3), fresh(3), 16, None),
    lambda m: m.allgather(fresh(70), fresh(70), 16, None),                          # more than fits the stack
    lambda m: m.alltoall(fresh(2), fresh(2), [[1, 2], [3, 4]], None),
    lambda m: m.alltoall_inplace(fresh(4), 16, None),
    lambda m: m.broadcast(Block(), fresh(3), 16, None),
    lambda m: m.batch_copy(((Block(), Block(), 5) for _ in range(3)), None),
    lambda m: m.token_dispatch(fresh(2), fresh(2), [2, 1], 16, np.zeros((3, 2), np.uint8), None),
    lambda m: m.token_dispatch_device(fresh(2), fresh(2), [2, 1], 16, Block(), None)])
def test_buffers_outlive_the_call(calls, call):
    """Buffers that only the argument refers to (made by an iterator) are alive, each at an address of its own, while
    the library runs, and given up afterwards."""
    m, _ = calls
    Block.live.clear()
    during = []
    m.bind([ctypes.cast(f, vp).value for f in watchers(m, during)])
    assert call(m) == -5
    (used, live), = during
    assert len(set(used)) == len(used) and set(used) <= live
    assert not Block.live


_watchers = []


def watchers(m, during):
    """Entry points that note the addresses they are given and what is alive at that time."""
    def words(p, n):
        return [ctypes.cast(p, ctypes.POINTER(u64))[i] for i in range(n)]

    args = {
        "dl_allgather": ([vp, vp, ctypes.c_int, sz, vp], lambda i, o, W, b, s: words(i, W) + words(o, W)),
        "dl_alltoall": ([vp, vp, ctypes.c_int, vp, vp], lambda i, o, W, c, s: words(i, W) + words(o, W)),
        "dl_alltoall_inplace": ([vp, ctypes.c_int, sz, vp], lambda b, W, c, s: words(b, W)),
        "dl_broadcast": ([vp, vp, ctypes.c_int, sz, vp], lambda a, d, k, b, s: [a] + words(d, k)),
        "dl_batch_copy": ([vp, sz, vp], lambda p, n, s: [words(p, 3 * n)[3 * i + q] for i in range(n) for q in (0, 1)]),
        "dl_token_dispatch": ([vp, vp, ctypes.c_int, vp, sz, vp, vp], lambda i, o, W, t, r, d, s: words(i, W) + words(o, W)),
        "dl_token_dispatch_device": ([vp, vp, ctypes.c_int, vp, sz, vp, vp], lambda i, o, W, t, r, d, s: words(i, W) + words(o, W) + [d]),
    }

    def watch(f):
        def g(*a):
            during.append((f(*a), set(Block.live)))
            return -5
        return g

    _watchers[:] = [ctypes.CFUNCTYPE(ctypes.c_int, *args[n][0])(watch(args[n][1])) if n in args else ctypes.CFUNCTYPE(ctypes.c_int)(lambda: -5)
                    for n in m.NAMES]
    return _watchers


@pytest.mark.parametrize("form", [lambda m: m, lambda m: m.tolist(), lambda m: m.astype(np.int64), np.asfortranarray, lambda m: iter(m.tolist()),
                                  lambda m: np.repeat(m, 2, axis=1)[:, ::2]])
@pytest.mark.parametrize("buffers", [iter, list])
def test_any_form_of_mask_with_iterators_for_the_buffers(calls, form, buffers):
    """Whatever form the mask has, the buffers may come from iterators, which can be read once only."""
    m, seen = calls
    mask = np.array([[3, 0], [0, 1], [5, 7]], dtype=np.uint8)
    with pytest.raises(binding.DlError):                                            # (the stub's -5)
        binding.dl_token_dispatch(buffers([1, 2]), buffers([3, 4]), [2, 1], 16, form(mask), 9)
    (got,) = seen
    assert got[:6] == ("dl_token_dispatch", [1, 2], [3, 4], [2, 1], 16, got[5]) and got[6] == 9
    assert [v != 0 for v in got[7]] == (mask != 0).ravel().tolist()


def test_token_counts_are_a_sequence(calls):
    m, seen = calls
    for mask in (bytes(6), [[0, 1]] * 3):
        with pytest.raises(TypeError):
            binding.dl_token_dispatch([1, 2], [3, 4], iter([2, 1]), 16, mask, None)
    assert not seen


def test_dispatch_of_unlikely_counts_and_ranks(calls):
    """Counts beyond 32 bits do not match a mask that their remainders would; any number of ranks reaches the library."""
    m, seen = calls
    with pytest.raises(ValueError):
        m.token_dispatch([1, 2], [3, 4], [2 ** 32 + 2, 1], 16, np.zeros((3, 2), np.uint8), None)
    assert not seen
    W = list(range(1, 71))
    assert m.token_dispatch(W, W, [1] * 70, 16, np.ones((70, 70), np.uint8), None) == -5
    assert m.token_dispatch_device(W, W, [1] * 70, 16, 2 ** 62, None) == -5
    assert [c[1:5] for c in seen] == [(W, W, [1] * 70, 16)] * 2


@pytest.mark.parametrize("bad", ["0", 1.0, 1.9, b"1", (1,), np.float64(2.0)])
def test_modes_and_tickets_are_whole_numbers(calls, bad):
    """What is no whole number is refused, not converted; ctypes' own integers are taken as by the entry points."""
    m, seen = calls
    for call in (binding.dl_set_mode, binding.dl_trigger, binding.dl_wait, lambda v: binding.dl_wait(1, v)):
        with pytest.raises(ctypes.ArgumentError):
            call(bad)
    assert not seen
    for f, args in ((m.set_mode, (1,)), (m.trigger, (2,)), (m.wait, (3, 4))):
        assert f(*args) == -5 and f(*(np.int32(a) for a in args)) == -5 and f(True, *args[1:]) == -5
        assert f(ctypes.c_int(1), *args[1:]) is NotImplemented
    assert [c[1] for c in seen] == [1, 1, 1, 2, 2, 1, 3, 3, 1]
    with pytest.raises(binding.DlError):                                            # the library's own refusal: taken as 1 << 20
        binding.dl_set_mode(ctypes.c_int(1 << 20))


def test_an_attribute_error_inside_data_ptr_is_the_callers_to_see(calls):
    """It does not turn the object into a number (a one-element tensor's value is not its address)."""
    m, seen = calls

    class Lost:
        def data_ptr(self):
            return self.storage

        def __index__(self):
            return 7

    for call in (lambda: m.allgather([Lost()], [1], 1, None), lambda: m.broadcast(Lost(), [1], 1, None),
                 lambda: m.batch_copy([(1, Lost(), 3)], None), lambda: m.token_dispatch_device([1], [2], [1], 1, Lost(), None)):
        with pytest.raises(AttributeError, match="storage"):
            call()
    assert not seen


def test_the_calls_made_with_ctypes_objects(calls, monkeypatch):
    """marshal_ctypes.py, for a Python without the extension, hands the entry points the same."""
    from types import SimpleNamespace

    from paper_2511_06605_amd import marshal_ctypes
    m, seen = calls
    monkeypatch.setattr(binding, "_lib", SimpleNamespace(**stubs))
    B = [Tensor(2 ** 63), 1, 2, 3]
    descs = [(0x10, Tensor(0x20), 3), [Tensor(5), None, np.int32(9)]]
    mask = np.array([[3, 0], [0, 1], [5, 7]], dtype=np.uint8)
    table = [("allgather", lambda: (iter(A), iter(B), np.int64(4096), Stream())), ("allgather", lambda: ([], [], 0, None)),
             ("alltoall", lambda: ([8, 9], [10, 11], [[1, 2], [3, 2 ** 40]], 3)), ("alltoall_inplace", lambda: (iter(A), 2 ** 33, 4)),
             ("broadcast", lambda: (Tensor(0x99), iter(A), 1, None)), ("batch_copy", lambda: (iter(descs), 5)),
             ("batch_copy_static", lambda: (descs, 5)), ("batch_swap", lambda: (descs, None)),
             ("token_dispatch", lambda: (iter([1, 2]), iter([3, 4]), [2, 1], 16, mask != 0, 9)),
             ("token_dispatch_device", lambda: (iter([1, 2]), iter([3, 4]), [2, 1], 16, Tensor(2 ** 62), 9)),
             ("set_mode", lambda: (3,)), ("trigger", lambda: (2 ** 64 - 1,)), ("wait", lambda: (3, 4))]
    for name, args in table:
        assert getattr(m, name)(*args()) == -5 and getattr(marshal_ctypes, name)(*args()) == -5
        native, other = seen[-2:]
        if name == "token_dispatch":  # the address of the mask is its own
            native, other = ([v for q, v in enumerate(c) if q != 5] for c in (native, other))
        assert native == other, name
    assert m.last_ticket() == marshal_ctypes.last_ticket()
    assert {n[3:] for n in stubs} <= set(dir(marshal_ctypes))
    with pytest.raises(ValueError):
        marshal_ctypes.allgather([1], [1, 2], 1, None)


def test_the_library_is_built_where_python_has_no_headers(tmp_path, monkeypatch, capsys):
    """The library first, whatever becomes of the extension; no headers or no C compiler: the library alone."""
    from paper_2511_06605_amd import build as b
    ran = []
    monkeypatch.setattr(b, "_run", lambda cmd, verbose: ran.append(cmd))
    monkeypatch.setattr(b, "HERE", str(tmp_path))
    monkeypatch.setattr(b, "MARSHAL", str(tmp_path / "_marshal.so"))
    assert b.build() == b.LIB
    assert [c[-1] for c in ran] == [b.LIB, b.MARSHAL]
    ran.clear()
    monkeypatch.setattr(b.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert b.build() == b.LIB
    assert [c[-1] for c in ran] == [b.LIB] and "headers" in capsys.readouterr().err


def test_without_the_extension_the_package_uses_ctypes(monkeypatch):
    from paper_2511_06605_amd import marshal_ctypes
    import paper_2511_06605_amd
    import sys
    monkeypatch.setitem(sys.modules, "paper_2511_06605_amd._marshal", None)         # import raises ImportError
    monkeypatch.delattr(paper_2511_06605_amd, "_marshal", raising=False)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_marshal", None)
    assert binding._native() is marshal_ctypes and binding._lib is not None
    assert binding.dl_last_ticket() == 0


# Python.h includes longintrepr.h from 3.10 on and by another name from 3.11; a Python may be built with digits of 15 bits; from
# 3.12 on an int lies differently
@pytest.mark.parametrize("minor,bits,in_place", [(9, 30, True), (10, 30, True), (10, 15, False), (11, 30, True), (11, 15, False), (12, 30, False)])
def test_builds_for_other_pythons(tmp_path, minor, bits, in_place):
    here = sysconfig.get_paths()["include"]
    cc = next(filter(None, map(shutil.which, ("gcc", "cc"))), None)
    if not cc or sysconfig.get_python_version() != "3.10" or not os.path.exists(os.path.join(here, "longintrepr.h")):
        pytest.skip("needs a C compiler and the headers of Python 3.10, from which the others are made")
    inc = tmp_path / "include"
    shutil.copytree(here, inc)

    def edit(name, pattern, by):
        text, n = re.subn(pattern, by, (inc / name).read_text())
        assert n == 1, (name, pattern)
        (inc / name).write_text(text)

    edit("patchlevel.h", r"(#define PY_MINOR_VERSION\s+)\d+", rf"\g<1>{minor}")
    if minor < 10:
        edit("Python.h", r'#include "longintrepr.h"\n', "")
    if minor > 10:
        edit("Python.h", r'#include "longintrepr.h"', '#include "cpython/longintrepr.h"')
        shutil.move(inc / "longintrepr.h", inc / "cpython" / "longintrepr.h")
    probe = tmp_path / "probe.c"
    probe.write_text(f'#include "{os.path.join(build.CSRC, "dl_marshal.c")}"\n'
                     f'_Static_assert((PY_VERSION_HEX >> 16 & 0xFF) == {minor} && PLAIN_INTS == {int(in_place)}, "which Pythons are read in place");\n')
    r = subprocess.run([cc, "-std=c11", "-fsyntax-only", "-Wall", f"-DPYLONG_BITS_IN_DIGIT={bits}", "-I" + str(inc), str(probe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
