"""csrc/call.c: what reaches the library's functions, seen by stand-ins for them."""
import ctypes as C

import numpy as np
import pytest

import paper_2404_07947_amd as exe
from paper_2404_07947_amd import binding

vp, i32, ip = C.c_void_p, C.c_int32, C.POINTER(C.c_int32)


@pytest.fixture()
def call():
    exe.lib()
    return binding._call


def _at(f):
    return C.cast(f, vp).value


def _list(p, n):
    return [p[i] for i in range(n)] if p else None


@pytest.mark.parametrize("n", [1, 3, 1000])
def test_arguments(call, n):
    seen = {}

    def decode(model, count, ids, toks, lens, hidden, nxt, out):
        seen["decode"] = (model, count, _list(ids, n), _list(toks, n), _list(lens, n), hidden, out)
        for i in range(n):
            nxt[i] = 7 + i
        return 5

    def encode(model, count, ids, lens, toks, res, hidden, nxt, out):
        seen["encode"] = (model, count, _list(ids, n), _list(lens, n), _list(toks, 2 * n), _list(res, n), hidden, bool(nxt), out)
        return -3

    def release(model, count, ids):
        seen["release"] = (model, count, _list(ids, n))
        return 0

    d = C.CFUNCTYPE(i32, vp, i32, ip, ip, ip, vp, ip, vp)(decode)
    e = C.CFUNCTYPE(i32, vp, i32, ip, ip, ip, ip, vp, ip, vp)(encode)
    r = C.CFUNCTYPE(i32, vp, i32, ip)(release)
    ids, toks, two = np.arange(n, dtype=np.int32), np.arange(n, dtype=np.int32) * 3, np.arange(2 * n, dtype=np.int32)
    lens = np.ascontiguousarray(np.broadcast_to(np.int32(9), (n,)))
    lens.setflags(write=False)                                   # arguments may be read-only, results not
    nxt = np.zeros(n, dtype=np.int32)
    big = (1 << 63) + 16                                         # a pointer's upper half
    assert call.decode_step(_at(d), 4096, ids, toks, lens, None, nxt, big) == 5
    assert seen["decode"] == (4096, n, ids.tolist(), toks.tolist(), [9] * n, None, big)
    assert nxt.tolist() == list(range(7, 7 + n))
    assert call.encode(_at(e), 4096, ids, lens, two, None, 64, None, None) == -3
    assert seen["encode"] == (4096, n, ids.tolist(), [9] * n, two.tolist(), None, 64, False, None)
    assert call.seq_release(_at(r), None, ids) == 0 and seen["release"] == (None, n, ids.tolist())


def test_refuses(call):
    ids = np.arange(4, dtype=np.int32)
    frozen = ids.copy()
    frozen.setflags(write=False)
    @C.CFUNCTYPE(i32, vp, i32, ip)
    def never(model, count, p):
        raise AssertionError

    bad = [np.arange(4, dtype=np.int64), np.arange(8, dtype=np.int32)[::2], [1, 2], 3, np.arange(4, dtype=np.float32),
           np.arange(4, dtype=np.uint32), np.arange(4, dtype=">i4")]
    for b in bad:
        with pytest.raises((TypeError, ValueError, BufferError)):
            call.seq_release(_at(never), 4096, b)
    with pytest.raises((TypeError, ValueError, BufferError)):
        call.decode_step(_at(never), 4096, ids, ids, ids, None, frozen, None)
    with pytest.raises(TypeError):
        call.decode_step(_at(never), 4096, ids)
    with pytest.raises(TypeError):
        call.decode_step(_at(never), 4096, ids, ids, ids, "x", None, None)
    with pytest.raises(ValueError):
        call.seq_release(None, 4096, ids)


@pytest.mark.parametrize("ids", [[0, 1], (0, 1), np.arange(2), np.arange(4, dtype=np.int32)[::2], 3])
def test_forms_of_a_call(call, ids):
    """Model converts what it is given, as before: the library is reached and refuses the null model."""
    m = object.__new__(exe.Model)
    m._h = None
    for f in (lambda: m.decode_step(ids, ids, ids), lambda: m.encode(ids, ids), lambda: m.seq_release(ids)):
        with pytest.raises(exe.ExeError, match="null model"):
            f()


@pytest.mark.parametrize("want", [True, False])
def test_a_call_without_ids(want):
    """None for the ids is a TypeError, whatever else is given: the number of sequences is theirs."""
    exe.lib()
    m = object.__new__(exe.Model)
    m._h = None
    one = np.ones(1, dtype=np.int32)
    for f in (lambda: m.encode(None, one, want_tokens=want), lambda: m.decode_step(None, one, one, want_tokens=want),
              lambda: m.seq_release(None)):
        with pytest.raises(TypeError):
            f()


def test_the_extension_is_the_interpreters_own(call, monkeypatch):
    """Built against one Python's headers, loaded by that Python: another one in the same tree is told to build its own."""
    import sysconfig
    assert call.__file__.endswith("_call" + sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(sysconfig, "get_config_var", lambda name: ".cpython-399-none.so")
    with pytest.raises(ImportError, match="cpython-399"):
        exe.lib()
