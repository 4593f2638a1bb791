"""The C route of a decode step's two calls takes what the Python checks take and hands back the rest; through the binding
both routes raise the same errors.  On the CPU: objects that answer like device tensors, and a library whose entry points
only record their arguments."""
import ctypes as C
import os
import shutil
import types

import pytest
import torch

from paper_2512_17917_amd import binding as kvr
from paper_2512_17917_amd import build as B

P, I, L = C.c_void_p, C.c_int32, C.c_int64


class Fake(torch.Tensor):
    """Answers like a device tensor; a type by itself stands for any other type."""

    def __new__(cls, dtype, n, at, cuda=True, contiguous=True):
        t = torch.Tensor._make_subclass(cls, torch.empty(0))
        t._dtype, t._cuda, t._n, t._at, t._c = dtype, cuda, n, at, contiguous
        return t

    dtype = property(lambda self: self._dtype)
    is_cuda = property(lambda self: self._cuda)

    def element_size(self):
        return 1

    def is_contiguous(self):
        return self._c

    def numel(self):
        return self._n

    def data_ptr(self):
        return self._at


@pytest.fixture()
def fast():
    if not os.path.exists(B.FAST):
        pytest.skip("the extension was left out of the build")
    kvr.lib()
    m, got = kvr._fast, []
    assert m is not None
    step = C.CFUNCTYPE(I, P, P, P, P, P, P, P, I, P, L, I, I, P, P, P, I, P, P, I, P, P, P)(lambda *a: got.append(a) or 7)
    att = C.CFUNCTYPE(I, P, P, P, P, P, I, P, P, P, P, I, P, P, L, P, C.c_size_t, P, P)(lambda *a: got.append(a) or 9)
    types = (torch.float32, torch.bfloat16, torch.int32, torch.uint8, torch.Tensor)
    m.setup(C.cast(step, P).value, C.cast(att, P).value, *types)
    yield m, got
    real = kvr.lib()
    m.setup(C.cast(real.kvr_step_update, P).value, C.cast(real.kvr_attend_decode, P).value, *types)


def call(dt):
    """(desc, arguments of step_update, of attend_decode): B 2, 8 heads on 4, three rows of 5 slots."""
    d = kvr.make_desc(2, 8, 4, 3, 5, dt, seed=1)
    U, R, V, N, E = 8, 6, 11, 20, 4
    i32, f32 = torch.int32, torch.float32
    t = lambda k, ty, n: Fake(ty, n, 1000 + 16 * k)
    step = [t(0, dt, U * 128), t(1, dt, U * 128), t(2, i32, 2), t(3, dt, U * R * 128), t(4, dt, U * R * 128), t(5, i32, U * R), R,
            t(6, f32, U * N), N, 3, 2, t(7, i32, U * E), t(8, i32, U * E), t(9, i32, U), E, t(10, i32, U * V), t(11, i32, U), V,
            t(12, dt, U * 15 * 128), t(13, dt, U * 15 * 128)]
    att = [t(0, dt, 16 * 128), t(1, dt, U * R * 128), t(2, dt, U * R * 128), t(3, i32, U * R), R, t(4, dt, U * 15 * 128),
           t(5, dt, U * 15 * 128), t(6, i32, U * V), t(7, i32, U), V, t(8, f32, 16 * 128), t(9, f32, U * N), N, t(10, torch.uint8, 4096)]
    return d, step, att


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_arguments_arrive(fast, dt):
    m, got = fast
    d, step, att = call(dt)
    at = [x.data_ptr() if isinstance(x, Fake) else x for x in step]
    assert m.step_update(C.addressof(d), 77, *step) == 7
    assert list(got[-1]) == [C.addressof(d), *at, 77]
    at = [x.data_ptr() if isinstance(x, Fake) else x for x in att]
    assert m.attend_decode(C.addressof(d), 77, 55, *att) == 9
    assert list(got[-1]) == [C.addressof(d), *at, 4096, 55, 77]
    for k in (3, 5, 6, 7, 8, 11):                     # the tensors that may be absent
        less = list(att)
        less[k] = None
        assert m.attend_decode(C.addressof(d), 77, 0, *less) == 9 and got[-1][k + 1] is None


@pytest.mark.parametrize("which", [0, 1])
def test_every_check_refuses(fast, which):
    m, got = fast
    dt = torch.bfloat16
    d, *both = call(dt)
    run = [lambda a: m.step_update(C.addressof(d), 0, *a), lambda a: m.attend_decode(C.addressof(d), 0, 0, *a)][which]
    good = both[which]
    assert run(good) is not None
    n = len(got)
    none_ok = [(15, 16), (3, 5, 6, 7, 8, 11)][which]
    for k, x in enumerate(good):
        if isinstance(x, Fake):
            other = torch.float16
            bad = [Fake(other, x._n, x._at), Fake(x.dtype, x._n, x._at, cuda=False), Fake(x.dtype, x._n, x._at, contiguous=False), 3, "x"]
            if x.dtype != torch.uint8:
                bad.append(Fake(x.dtype, x._n - 1, x._at))
            if k not in none_ok:
                bad.append(None)
        else:
            bad = [None, 1.5, "x", 1 << 70]
        for b in bad:
            assert run(good[:k] + [b] + good[k + 1:]) is None, (k, b)
    assert run(good[:-1]) is None and len(got) == n


# --- through the binding ------------------------------------------------------------------------------------------------
class Other(C.Structure):
    """Not the options, not the descriptor."""
    _fields_ = [("x", C.c_int32)]


class Alike(C.Structure):
    """The descriptor's fields under another name."""
    _fields_ = kvr.kvr_desc._fields_


class Sub(kvr.kvr_desc):
    pass


@pytest.fixture()
def routes(fast, monkeypatch):
    """run(name, desc, *args) -> [(what came out of the call, recorded arguments) of the C route, of the Python route]"""
    m, got = fast
    real = kvr.lib()
    take = lambda a: got.append([C.addressof(x.contents) if isinstance(x, C._Pointer) and x else
                                 None if isinstance(x, C._Pointer) else x for x in a]) or 0
    entry = lambda f: C.CFUNCTYPE(f.restype, *f.argtypes)(lambda *a: take(a))      # checks its arguments as the library's does
    e = {n: entry(getattr(real, n)) for n in ("kvr_step_update", "kvr_attend_decode")}
    m.setup(*(C.cast(e[n], P).value for n in e), torch.float32, torch.bfloat16, torch.int32, torch.uint8, torch.Tensor)
    stand_in = types.SimpleNamespace(**e)

    def run(name, *args, **more):
        came = []
        for route in (m, None):
            del got[:]
            with monkeypatch.context() as p:
                p.setattr(kvr, "_lib", stand_in)
                p.setattr(kvr, "_stream", lambda: 77)
                p.setattr(kvr, "_fast", route)
                try:
                    came.append((getattr(kvr, name)(*args, **more), list(got)))
                except Exception as x:
                    assert not got
                    came.append((type(x), str(x)))
        return came
    return run


def test_types_of_the_structures(routes):
    """A structure of another type, a pointer or a number in place of the descriptor or the options is refused by both."""
    d, step, att = call(torch.bfloat16)
    o = kvr.kvr_attend_opts()
    for opts in (None, o):
        c, py = routes("kvr_attend_decode", d, *att, opts=opts)
        assert c == py and len(c[1]) == 1
    c, py = routes("kvr_step_update", d, *step)
    assert c == py and len(c[1]) == 1
    sub = Sub.from_buffer_copy(bytes(d))
    c, py = routes("kvr_step_update", sub, *step)
    assert c == py and len(c[1]) == 1
    for bad in (d, C.c_int(5), Other(), C.pointer(o), C.byref(o), 5, "x"):
        c, py = routes("kvr_attend_decode", d, *att, opts=bad)
        assert c == py and issubclass(c[0], (C.ArgumentError, TypeError)), (bad, c, py)
    for bad in (o, C.c_int(5), Other(), Alike.from_buffer_copy(bytes(d)), C.pointer(d), 5, None):
        for name, args in (("kvr_step_update", step), ("kvr_attend_decode", att)):
            c, py = routes(name, bad, *args)
            assert c == py and issubclass(c[0], (C.ArgumentError, TypeError, AttributeError)), (bad, c, py)


class NoTensor:
    """Answers like a tensor and is none."""

    def __init__(self, t):
        self.dtype, self.is_cuda = t.dtype, t.is_cuda
        self.is_contiguous, self.numel, self.data_ptr, self.element_size = t.is_contiguous, t.numel, t.data_ptr, t.element_size


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_every_argument_by_both_routes(routes, dt):
    """Each argument of each call replaced by what it must not be: the same error by both routes."""
    d, step, att = call(dt)
    for name, args in (("kvr_step_update", step), ("kvr_attend_decode", att)):
        for k, x in enumerate(args):
            if isinstance(x, Fake):
                bad = [Fake(torch.float16, x._n, x._at), Fake(x.dtype, x._n, x._at, cuda=False),
                       Fake(x.dtype, x._n, x._at, contiguous=False), Fake(x.dtype, x._n - 1, x._at), NoTensor(x), None, 3, "x"]
            else:
                bad = [None, 1.5, "x", -1, True]
            for b in bad:
                c, py = routes(name, d, *args[:k], b, *args[k + 1:])
                assert c == py, (name, k, b if not isinstance(b, Fake) else (b._dtype, b._n))


def test_sizes_whose_products_wrap(routes):
    """Counts and descriptors whose products leave 64 bits (some come back as 0): refused as by the Python checks."""
    d, step, att = call(torch.bfloat16)
    for name, args, counts in (("kvr_step_update", step, (6, 8, 14, 17)), ("kvr_attend_decode", att, (4, 9, 12))):
        for k in counts:
            for n in (1 << 31, 1 << 54, 1 << 57, 1 << 61, 1 << 62, (1 << 63) - 1, 1 << 64):
                c, py = routes(name, d, *args[:k], n, *args[k + 1:])
                assert c == py and c[0] is ValueError, (name, k, n, c, py)
        for fields in (dict(batch=1 << 30, n_kv_heads=1 << 30), dict(w=1 << 30, head_dim=1 << 30), dict(r=1 << 28, w=1 << 28),
                       dict(batch=1 << 30, n_q_heads=1 << 30), dict(head_dim=1 << 30)):
            x = kvr.kvr_desc.from_buffer_copy(bytes(d))
            for f, v in fields.items():
                setattr(x, f, v)
            c, py = routes(name, x, *args)
            assert c == py and c[0] is ValueError, (name, fields, c, py)


# --- the build ----------------------------------------------------------------------------------------------------------
def test_build_leaves_the_extension_out(tmp_path, monkeypatch, capsys):
    """Without a compiler or Python.h: a message, no extension (nor a stale one), and a binding that calls through ctypes."""
    name = os.path.basename(B.FAST)
    assert B.FAST == kvr.FAST_PATH and name.startswith("_kvr_fast.") and name.count(".") == 2        # _kvr_fast.<interpreter>.so
    monkeypatch.setattr(B, "FAST", str(tmp_path / name))
    none = tmp_path / "empty"
    none.mkdir()
    for cc, include in ((str(tmp_path / "no-such-compiler"), None), ("gcc", str(none))):
        open(B.FAST, "w").write("from before")
        with monkeypatch.context() as p:
            p.setattr(B, "CC", cc)
            if include:
                p.setattr(B.sysconfig, "get_paths", lambda: {"include": include})
            assert B.build_fast() is False
        assert not os.path.exists(B.FAST) and "left out" in capsys.readouterr().err
    (tmp_path / "_kvr_fast.so").write_text("another interpreter's")
    monkeypatch.setattr(kvr, "FAST_PATH", B.FAST)
    monkeypatch.setattr(kvr, "_fast", None)
    kvr._load_fast(kvr.lib())
    assert kvr._fast is None
    if shutil.which(B.CC) and os.path.exists(os.path.join(B.sysconfig.get_paths()["include"], "Python.h")):
        assert B.build_fast() is True and os.path.exists(B.FAST)
