"""The binding's native calls against its own way through ctypes: the same arguments reach the library and the same results come back,
whatever form they are given in; with the library's calls replaced, so that this needs no GPU."""
import ctypes as C
import sysconfig

import numpy as np
import pytest

from paper_2502_18554_amd import binding as b

vp, sz, u, i = C.c_void_p, C.c_size_t, C.c_uint, C.c_int


class Tensor:
    def __init__(self, at, elements):
        self.at, self.elements = at, elements

    def data_ptr(self):
        return self.at

    def numel(self):
        return self.elements

    @property
    def nbytes(self):
        return 4 * self.elements


def _list(p, k):
    return [C.cast(p, C.POINTER(sz))[j] for j in range(k)]


@pytest.fixture
def seen(monkeypatch):
    """What the library's calls were given, by either way; every call answers 6 and, where asked, 777 (and 100, 101, ... per stream)."""
    L = b.lib()
    if b._native is None:
        pytest.skip("the native calls are not built")
    got = []

    def fill(p, n=1, v=777):
        for j in range(n if p else 0):
            C.cast(p, C.POINTER(sz))[j] = v + j

    def compress(d, n, eb, out, cap, size, ws, wb, st, fl):
        got.append(("compress", d, n, eb, out, cap, bool(size), ws, wb, st, fl))
        fill(size)
        return 6

    def decompress(d, n, out, cap, size, ws, wb, st, fl):
        got.append(("decompress", d, n, out, cap, bool(size), ws, wb, st, fl))
        fill(size)
        return 6

    def reduce(ch, by, k, op, out, cap, size, ws, wb, st, fl):
        got.append(("reduce", _list(ch, k), _list(by, k), k, op, out, cap, bool(size), ws, wb, st, fl))
        fill(size)
        return 6

    def step(d, n, loc, nl, op, out, cap, size, ws, wb, st, fl):
        got.append(("step", d, n, loc, nl, op, out, cap, bool(size), ws, wb, st, fl))
        fill(size)
        return 6

    def many(ch, by, k, outs, caps, ns, ws, wb, st, fl):
        got.append(("many", _list(ch, k), _list(by, k), k, _list(outs, k), _list(caps, k), bool(ns), ws, wb, st, fl))
        fill(ns, k, 100)
        return 6

    protos = (C.CFUNCTYPE(i, vp, sz, C.c_float, vp, sz, vp, vp, sz, vp, u), C.CFUNCTYPE(i, vp, sz, vp, sz, vp, vp, sz, vp, u),
              C.CFUNCTYPE(i, vp, vp, i, i, vp, sz, vp, vp, sz, vp, u), C.CFUNCTYPE(i, vp, sz, vp, sz, i, vp, sz, vp, vp, sz, vp, u),
              C.CFUNCTYPE(i, vp, vp, i, vp, vp, vp, vp, sz, vp, u))
    keep = [p(f) for p, f in zip(protos, (compress, decompress, reduce, step, many))]

    class Fake:
        zc_compress_ex, zc_decompress_ex, zc_reduce_compressed_op, zc_reduce_step_op, zc_decompress_many = keep

        @staticmethod
        def zc_compress(*a):
            return Fake.zc_compress_ex(*a, 0)

        @staticmethod
        def zc_decompress(*a):
            return Fake.zc_decompress_ex(*a, 0)

        @staticmethod
        def zc_reduce_compressed(ch, by, k, *a):
            return Fake.zc_reduce_compressed_op(ch, by, k, 0, *a, 0)

        @staticmethod
        def zc_reduce_compressed_ex(ch, by, k, *a):
            return Fake.zc_reduce_compressed_op(ch, by, k, 0, *a)

        @staticmethod
        def zc_reduce_step(d, n, loc, nl, *a):
            return Fake.zc_reduce_step_op(d, n, loc, nl, 0, *a, 0)

    native = b._native
    native.setup(*(C.cast(f, vp).value for f in keep), lambda: 3, lambda device: 0x5000 + device)
    monkeypatch.setattr(b, "_stream", lambda s=None: s.cuda_stream if s is not None else 0x5003)
    monkeypatch.setattr(b, "_lib", Fake)
    monkeypatch.setattr(b.C, "byref", lambda o: C.cast(C.pointer(o), vp))
    yield got
    monkeypatch.undo()
    b._load_native(L)


X, Y, Z, W = Tensor(0x1000, 10), Tensor(0x2000, 20), Tensor(0x3000, 30), Tensor(0x4000, 40)
STREAM = type("S", (), {"cuda_stream": 0x77})()
CALLS = [
    lambda **o: b.zc_compress(X, 10, 0.25, Y, W, **o),
    lambda **o: b.zc_compress(None, 0, 1e-3, Y, W, **o),
    lambda **o: b.zc_compress(X, 1 << 31, 3.0000000001, Y, W, out_cap=7, **o),
    lambda **o: b.zc_decompress(X, 33, Y, W, **o),
    lambda **o: b.zc_decompress(X, 33, None, W, **o),
    lambda **o: b.zc_decompress(X, 33, Y, W, out_cap_elems=3, **o),
    lambda **o: b.zc_reduce_step(X, 33, Z, 30, Y, W, **o),
    lambda **o: b.zc_reduce_step_op(X, np.int64(33), Z, np.int32(30), 2, Y, W, **o),
    lambda **o: b.zc_reduce_compressed([X, Z], [11, 12], Y, W, **o),
    lambda **o: b.zc_reduce_compressed_op((X, Z, X), (11, 12, 13), 1, Y, W, out_cap=5, **o),
    lambda **o: b.zc_reduce_compressed_op([X, Z], np.array([11, 12]), 2, Y, W, **o),
    lambda **o: b.zc_reduce_compressed([X, Z], [11], Y, W, **o),
    lambda **o: b.zc_decompress_many([X, Z], [11, 12], [Y, W], W, **o),
    lambda **o: b.zc_decompress_many([X], [11], [Y], W, out_cap_elems=[9], **o),
    lambda **o: b.zc_decompress_many([X] * 64, [11] * 64, [Y] * 64, W, **o),
    lambda **o: b.zc_decompress_many([X], [np.int64(11)], [Y], W, **o),
    lambda **o: b.zc_compress(X, np.int32(10), np.float32(0.25), Y, W, **o),
    lambda **o: b.zc_compress(X, 10, 1, Y, W, out_cap=np.int64(7), **o),
    lambda **o: b.zc_decompress(X, np.uint64(33), Y, W, out_cap_elems=np.int64(3), **o),
]


@pytest.mark.parametrize("call", range(len(CALLS)))
@pytest.mark.parametrize("options", [{}, {"sync": False}, {"sync": 1, "flags": 3}, {"stream": STREAM}, {"sync": False, "flags": 1}])
def test_both_ways_are_alike(seen, monkeypatch, call, options):
    native = CALLS[call](**options)
    monkeypatch.setattr(b, "_native", None)
    plain = CALLS[call](**options)
    assert native == plain and native[0] == 6
    assert len(seen) == 2 and seen[0] == seen[1]


# what the native calls leave to ctypes: by number in CALLS (an array of sizes, a list that is too short, numpy's numbers in a list)
DECLINED = {10, 11, 15}


@pytest.mark.parametrize("call", range(len(CALLS)))
@pytest.mark.parametrize("options", [{}, {"sync": False}, {"sync": 1, "flags": 3}, {"stream": STREAM}, {"sync": False, "flags": 1}])
def test_which_way_a_call_goes(seen, monkeypatch, call, options):
    """The plain forms are answered by the native calls, the others are declined ahead of any call of the library."""
    native, answers = b._native, []

    class Listening:
        def __getattr__(self, name):
            def listen(*args):
                before = len(seen)
                r = getattr(native, name)(*args)
                answers.append(r)
                assert len(seen) == before + (r is not NotImplemented)
                return r
            return listen

    monkeypatch.setattr(b, "_native", Listening())
    assert CALLS[call](**options)[0] == 6
    assert len(answers) == 1 and len(seen) == 1
    assert (answers[0] is NotImplemented) == (call in DECLINED)


def test_what_neither_takes(seen):
    with pytest.raises(AttributeError):
        b.zc_compress(X, 10, 0.25, Y, None)
    with pytest.raises(AttributeError):
        b.zc_decompress(7, 10, Y, W)
    with pytest.raises((TypeError, C.ArgumentError)):
        b.zc_compress(X, 10.0, 0.25, Y, W)
    with pytest.raises((TypeError, C.ArgumentError)):
        b.zc_compress(X, 10, "0.25", Y, W)
    with pytest.raises(AttributeError):
        b.zc_compress(X, 10, 0.25, Y, W, stream=7)
    with pytest.raises(IndexError):
        b.zc_reduce_compressed([X], [1, 2], Y, W)
    assert not seen


def test_native_calls_of_another_python(monkeypatch, tmp_path):
    """Native calls that were built for another Python are not looked at, and with some that do not load all calls go through ctypes, the first one
    as the later ones."""
    L = b.lib()
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert "-" in suffix                                   # (it names the Python)
    monkeypatch.setattr(b, "_HERE", str(tmp_path))
    monkeypatch.setattr(b, "_native", None)
    for name in ("_zc_calls.so", "_zc_calls" + suffix.replace("cpython-3", "cpython-4"), "_zc_calls" + suffix):
        (tmp_path / name).write_bytes(b"built elsewhere")
        monkeypatch.setattr(b, "_lib", None)
        assert b.lib() is not None and b._native is None
        assert b.zc_strerror(0) == L.zc_strerror(0).decode()


def test_build_without_python_headers(monkeypatch, tmp_path):
    """The library is built ahead of the native calls, and also where those cannot be."""
    from paper_2502_18554_amd import build
    ran = []
    calls = tmp_path / "_zc_calls.so"
    monkeypatch.setattr(build, "CALLS", str(calls))
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, check: ran.append(cmd[0]))
    build.build()
    assert ran == ["hipcc", "g++"]
    ran.clear()
    calls.write_bytes(b"of other sources")
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build() == build.LIB
    assert ran == ["hipcc"] and not calls.exists()
