"""The calls made from native code hand the C entry points what the binding functions hand them, over all forms of the
arguments that either accepts, and refuse what those refuse."""
import copy
import ctypes
import functools
import importlib.machinery
import inspect
import itertools
import os
import pickle
import shutil
import weakref

import pytest

import paper_2510_20111_amd as hzp
from paper_2510_20111_amd import binding as bd

NAMES = ["hzp_reduce_shard", "hzp_adamw_shard", "hzp_adamw_shard_dev", "hzp_gather_layer", "hzp_gather_layer_static",
         "hzp_gather_shard", "hzp_gather_layers", "hzp_gather_tensor"]


class Tensor:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


class Stream:
    cuda_stream = 0x7000


class Bad:
    def data_ptr(self):
        raise RuntimeError("no address")


class FakePlan:
    def __init__(self, address=0x1234560):
        self.handle = ctypes.c_void_p(address)


class Recorder:
    """Stands in for the library: every entry point notes its arguments, pointers to arrays as what they hold."""

    def __init__(self, status=0):
        self.got, self.status, self.keep = [], status, []
        for name in NAMES:
            real = getattr(bd._L, name)
            kinds = [ctypes.c_void_p if t not in (ctypes.c_uint32, ctypes.c_int, ctypes.c_float) else t for t in real.argtypes]
            fn = ctypes.CFUNCTYPE(ctypes.c_int, *kinds)(lambda *a, name=name: self.note(name, a))
            fn.argtypes = real.argtypes
            setattr(self, name, fn)

    def note(self, name, args):
        # (arrays are three words here; their addresses differ between two calls with lists, what they hold does not)
        held = {"hzp_reduce_shard": (5,), "hzp_adamw_shard": (6, 8, 9, 10, 11), "hzp_adamw_shard_dev": (6, 8, 9, 10, 11),
                "hzp_gather_layer": (4, 7), "hzp_gather_layer_static": (3, 5), "hzp_gather_shard": (4,), "hzp_gather_layers": (5, 7),
                "hzp_gather_tensor": (2,)}[name]
        out = []
        for i, a in enumerate(args):
            if i in held and a:
                out.append(list((ctypes.c_uint64 * 3).from_address(a)))
            elif name == "hzp_adamw_shard" and i == 5 and a:
                out.append(bytes((ctypes.c_char * ctypes.sizeof(bd.AdamW)).from_address(a)))
            else:
                out.append(a)
        self.got.append((name, out))
        return self.status


def pointers(base):
    words = [base, base + 0x100, base + 0x200]
    return [(ctypes.c_void_p * 3)(*words), (ctypes.c_uint64 * 3)(*words), list(words), tuple(words), [Tensor(w) for w in words],
            [words[0], Tensor(words[1]), words[2]]]


def addresses(a):
    return [a, Tensor(a), None, 0, (1 << 64) - 16]


STREAMS = [0, 0x55, (1 << 63) + 8, Stream()]
HYPER = bd.adamw_hyper(1e-3, 0.9, 0.95, 1e-8, 0.1, 0.25, 7)
CHOICES = {
    "plan": [FakePlan()], "layer": [3, 0, (1 << 32) - 1, True], "cls": [1], "level": [2, 1], "rank": [5], "j": [4], "tensor_id": [9],
    "layer_begin": [1], "layer_end": [6], "grad_slices": pointers(0x10000), "shard_ptrs": pointers(0x20000), "owner_ptrs": pointers(0x30000),
    "scale": [0.25, 1, 1e-60, float("inf")], "accumulate": [True, False, 1, 0, [], "yes"], "out_f32": addresses(0x4000), "R": [3, 0, 17],
    "grad_dtype": [0, 1, 2], "hyper": [HYPER], "scalars": addresses(0x5000), "master": pointers(0x60000), "m": pointers(0x70000),
    "v": pointers(0x80000), "param_out": [None] + pointers(0x90000), "bucket_out": None, "tensor_out": [None] + pointers(0xA0000),
    "shard_out": addresses(0x6000), "n_shards": [3, 2], "n_owners": [3, 64], "stream": STREAMS,
}


def forms(name):
    """Argument sets: a plain one, and it with each argument in each of its forms; by position and by name, defaults left out."""
    parameters = inspect.signature(getattr(bd, name)).parameters
    def choices(p):
        if p == "bucket_out":
            return pointers(0xB0000) if name == "hzp_gather_layers" else [None] + addresses(0x7000)
        if p == "tensor_out" and name == "hzp_gather_tensor":
            return addresses(0x8000)
        if p == "tensor_out" and name == "hzp_gather_layer_static":
            return [None] + pointers(0xA0000)
        if p in ("R", "n_shards", "n_owners") and parameters[p].default is None:
            return CHOICES[p] + [None]
        return CHOICES[p]
    plain = {p: choices(p)[0] for p in parameters}
    for p in parameters:
        for c in choices(p):
            yield dict(plain, **{p: c})
    short = {p: x for p, x in plain.items() if parameters[p].default is inspect.Parameter.empty}
    yield dict(short, stream=0x66)


def both(monkeypatch, name, args, kwargs, status=0):
    """(what the binding function did, what the native call did)"""
    native = getattr(bd, name)
    assert type(native).__name__ == "Call"
    out = []
    for side in (0, 1):
        rec = Recorder(status)
        monkeypatch.setattr(bd, "_L", Spy(rec, monkeypatch))
        entry = ctypes.cast(getattr(rec, name), ctypes.c_void_p).value
        call = native.__wrapped__ if side == 0 else bd._calls.Call(name, entry, native.__wrapped__, bd._check, ctypes.Array, ctypes.c_void_p, bd.AdamW)
        try:
            result = call(*args, **kwargs)
        except Exception as e:      # noqa: BLE001
            result = (type(e), str(e))
        out.append((result, rec.got))
        monkeypatch.undo()
    return out


class Spy:
    def __init__(self, rec, monkeypatch):
        self.rec, self.real = rec, bd._L

    def __getattr__(self, name):
        return getattr(self.rec, name) if name in NAMES else getattr(self.real, name)


@pytest.mark.parametrize("name", NAMES)
def test_native_calls_hand_over_what_the_binding_functions_do(monkeypatch, name):
    parameters = list(inspect.signature(getattr(bd, name)).parameters)
    n = 0
    for values in forms(name):
        given = [p for p in parameters if p in values]
        for by_position in {0, 1, len([p for p, q in zip(parameters, given) if p == q])}:
            args = [values[p] for p in given[:by_position]]
            kwargs = {p: values[p] for p in given[by_position:]}
            a, b = both(monkeypatch, name, args, kwargs)
            assert a == b, (args, kwargs)
            n += len(a[1])
    assert n > 20


@pytest.mark.parametrize("name", NAMES)
def test_native_calls_refuse_what_the_binding_functions_refuse(monkeypatch, name):
    parameters = inspect.signature(getattr(bd, name)).parameters
    plain = next(forms(name))
    plain["stream"] = 0x77
    wrong = [dict(plain, **{p: x}) for p, x in itertools.product(parameters, (Bad(), "text", 1.5, -1, 1 << 32, 1 << 70, b"x", object()))
             if not (p in ("stream",) and x is None)]
    wrong += [dict(plain, no_such_argument=1)] + [{q: x for q, x in plain.items() if q != p} for p in parameters
                                                  if parameters[p].default is inspect.Parameter.empty]
    for kwargs in wrong:
        a, b = both(monkeypatch, name, [], kwargs)
        if a[1]:    # taken, with the number or the bytes as they are: so does the native call
            assert len(b[1]) == 1 and a[0] == b[0], kwargs
            if not any(isinstance(x, bytes) for x in kwargs.values()):
                assert a == b, kwargs
        else:
            assert a == b, kwargs
    for args in ([], [1] * 20, list(plain.values()) + [1]):
        a, b = both(monkeypatch, name, args, {})
        assert a == b
    a, b = both(monkeypatch, name, list(plain.values())[:1], dict(plain))      # an argument twice
    assert a == b
    # a status of the library is the same exception
    a, b = both(monkeypatch, name, [], plain, status=hzp.HZP_ERR_RANGE)
    assert a == b and a[0][0] is hzp.HzpError


def test_native_calls_look_like_the_binding_functions():
    for name in NAMES:
        f = getattr(hzp, name)
        assert callable(f) and f.__name__ == name and f.__doc__ == f.__wrapped__.__doc__
        assert inspect.signature(f) == inspect.signature(f.__wrapped__)


def test_usual_calls_do_not_go_through_the_binding_functions():
    def not_this_way(*a, **k):
        raise AssertionError("went to the binding function")
    rec = Recorder()
    for name in NAMES:
        call = bd._calls.Call(name, ctypes.cast(getattr(rec, name), ctypes.c_void_p).value, not_this_way, bd._check, ctypes.Array,
                              ctypes.c_void_p, bd.AdamW)
        signature = inspect.signature(getattr(bd, name)).parameters
        values = next(forms(name))
        call(**values)
        call(*values.values())
        stream = {"stream": 0x99}
        call(*[x for p, x in values.items() if signature[p].default is inspect.Parameter.empty], **stream)
        for p, x in values.items():
            if isinstance(x, ctypes.Array):
                call(**dict(values, **{p: [Tensor(1 << 20), 1 << 21, Tensor(1 << 22)]}))
    assert len(rec.got) >= 4 * len(NAMES)


@pytest.mark.parametrize("name", NAMES)
def test_native_calls_behave_as_functions(name):
    """A program can hold, copy, send, wrap, annotate and bind them as it can the functions beside them."""
    f, plain = getattr(hzp, name), hzp.hzp_plan_free
    for g in (plain, f):
        for protocol in range(pickle.HIGHEST_PROTOCOL + 1):
            assert pickle.loads(pickle.dumps(g, protocol)) is g
        assert pickle.loads(pickle.dumps(functools.partial(g, 1))).func is g
        assert copy.copy(g) is g and copy.deepcopy({"call": [g]})["call"][0] is g
        assert weakref.ref(g)() is g
        assert inspect.isfunction(g) and inspect.isroutine(g) and callable(g) and isinstance(g, type(plain))
        assert repr(g).startswith("<function %s at 0x" % g.__name__)
        assert g == g and g != f.__wrapped__ and {g: 1}[g] == 1 and g.__eq__(g) is True
        g.mark = 5
        assert g.mark == 5 and vars(g)["mark"] == 5 and "mark" in dir(g)
        del g.mark
        assert not hasattr(g, "mark")
        with pytest.raises(AttributeError):
            del g.mark
        wrapped = functools.wraps(g)(lambda: None)
        assert wrapped.__name__ == g.__name__ and wrapped.__module__ == g.__module__

        class Holder:
            method = g
        holder = Holder()
        assert holder.method.__self__ is holder and holder.method.__func__ is g and Holder.method is g
        assert inspect.ismethod(holder.method) and inspect.ismethod(g.__get__(holder))


def test_other_defaults_are_used(monkeypatch):
    """A default that the program sets on the function counts, as it does for any function."""
    rec = Recorder()
    monkeypatch.setattr(bd, "_L", Spy(rec, monkeypatch))
    function = bd.hzp_gather_shard.__wrapped__
    call = bd._calls.Call("hzp_gather_shard", ctypes.cast(rec.hzp_gather_shard, ctypes.c_void_p).value, function, bd._check, ctypes.Array,
                          ctypes.c_void_p, bd.AdamW)
    args = (FakePlan(), 0, 0, 1, [1 << 20, 1 << 21, 1 << 22], 1 << 23)
    call(*args, stream=7)
    monkeypatch.setattr(call, "__defaults__", (9, 2))
    call(*args)
    monkeypatch.undo()
    call(*args, stream=7)
    assert [got[1][-1] for got in rec.got] == [7, 9, 7] and [got[1][5] for got in rec.got] == [3, 2, 3]


def test_calls_are_let_go():
    rec = Recorder()
    call = bd._calls.Call("hzp_gather_shard", ctypes.cast(rec.hzp_gather_shard, ctypes.c_void_p).value, lambda: None, bd._check,
                          ctypes.Array, ctypes.c_void_p, bd.AdamW)
    gone = weakref.ref(call)
    del call
    assert gone() is None
    with pytest.raises(TypeError):
        bd._calls.Call("hzp_gather_shard", 1, print, bd._check, ctypes.Array, ctypes.c_void_p, bd.AdamW)


class Counted(Tensor):
    """A tensor that counts how often its address was asked for, and may refuse to give it."""

    def __init__(self, address, error=None):
        super().__init__(address)
        self.asked, self.error = 0, error

    def data_ptr(self):
        self.asked += 1
        if self.error is not None:
            error, self.error = self.error, None        # the first time only
            raise error
        return self.address


def counted(name, n=3):
    """Arguments of a plain call, with tensors for all device buffers; and these tensors."""
    values = {p: x for p, x in next(forms(name)).items() if p != "stream"}
    tensors = []
    for p in values:
        if p in ("grad_slices", "shard_ptrs", "owner_ptrs", "master", "m", "v", "param_out") or (p == "bucket_out" and name == "hzp_gather_layers"):
            values[p] = [Counted((len(tensors) + 1 + i) << 12) for i in range(n)]
            tensors += values[p]
        elif p in ("out_f32", "scalars", "shard_out", "bucket_out"):
            values[p] = Counted(1 << 40)
            tensors.append(values[p])
    return values, tensors


def native(monkeypatch, name, function=None):
    """(recorder, the native call with it in the library's place)"""
    rec = Recorder()
    monkeypatch.setattr(bd, "_L", Spy(rec, monkeypatch))
    return rec, bd._native_call(function or getattr(bd, name).__wrapped__)


def elsewhere(name):
    def function(*args, **kwargs):
        raise AssertionError("went to the binding function")
    function.__name__ = name
    return function


@pytest.mark.parametrize("name", NAMES)
def test_the_current_stream_is_looked_up_in_native_calls(monkeypatch, name):
    """A call without a stream takes torch's current one, and asks every tensor for its address once."""
    monkeypatch.setattr("torch.cuda.current_stream", lambda: Stream())
    rec, call = native(monkeypatch, name, elsewhere(name))
    for extra in ({}, {"stream": None}):
        values, tensors = counted(name)
        call(**values, **extra)
        assert [t.asked for t in tensors] == [1] * len(tensors) and len(tensors) > 2
    assert [got[1][-1] for got in rec.got] == [Stream.cuda_stream] * 2


@pytest.mark.parametrize("name", NAMES)
def test_addresses_are_asked_for_once(monkeypatch, name):
    """Whatever sends a call to the binding function is seen before a tensor is asked: numbers of other types, longer lists, no stream
    (there is no GPU here: looking it up fails as it does in the binding function)."""
    rec, call = native(monkeypatch, name)
    def error(f, values):
        try:
            f(**values)
        except Exception as e:      # noqa: BLE001
            return type(e), str(e)
    monkeypatch.setattr("torch.cuda.current_stream", lambda: 1 // 0)
    got = []
    for f in (call, call.__wrapped__):
        values, tensors = counted(name)
        got.append((error(f, values), [t.asked for t in tensors]))
    assert got[0] == got[1] and got[0][0][0] is ZeroDivisionError and set(got[0][1]) == {1}
    parameters = inspect.signature(call).parameters
    others = [{}] + [{p: x} for p, x in (("scale", 1), ("accumulate", 1), ("cls", True), ("grad_dtype", True), ("n_shards", True), ("n_owners", True))
                     if p in parameters]
    for other in others:
        values, tensors = counted(name, 3 if other else 600)
        call(**dict(values, stream=7, **other) if not set(other) & set(values) else dict(values, stream=7) | other)
        assert [t.asked for t in tensors] == [1] * len(tensors), other
    assert len(rec.got) == len(others)
    for values in ({p: x for p, x in values.items() if p != "plan"}, dict(values, no_such_argument=1), dict(values, stream=object())):
        tensors = [t for x in values.values() if isinstance(x, list) for t in x]
        before = [t.asked for t in tensors]
        assert error(call, values)[0] in (TypeError, AttributeError)
        assert [t.asked for t in tensors] in (before, [n + 1 for n in before])


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("error", [KeyboardInterrupt, SystemExit, TimeoutError, RuntimeError, AttributeError])
def test_errors_of_the_arguments_are_not_lost(monkeypatch, name, error):
    """What an argument's own code raises ends the call, as it does in the binding function."""
    rec, call = native(monkeypatch, name)
    n = len(counted(name)[1])
    for at in range(n):
        for f in (call, call.__wrapped__):
            values, tensors = counted(name)
            tensors[at].error = error("at %d" % at)
            with pytest.raises(error, match="^at %d$" % at):
                f(**values, stream=7)
            assert [t.asked for t in tensors] == [1] * (at + 1) + [0] * (n - at - 1)
    values, tensors = counted(name)
    raising = type("S", (), {"cuda_stream": property(lambda self: (_ for _ in ()).throw(error("stream")))})()
    for f in (call, call.__wrapped__):
        with pytest.raises(error):
            f(**values, stream=raising)
    assert not rec.got


def test_only_a_module_built_for_this_interpreter_is_loaded(monkeypatch, tmp_path):
    """The module reads the interpreter's own structures, so one that was built for another must not be taken for it."""
    suffix = importlib.machinery.EXTENSION_SUFFIXES[0]
    assert "cpython" in suffix and bd._calls.__file__.endswith(os.sep + "_calls" + suffix)
    monkeypatch.setattr(bd, "_HERE", str(tmp_path))
    for other in ("_calls.so", "_calls.cpython-399-x86_64-linux-gnu.so", "_calls.abi3.so"):
        (tmp_path / other).write_bytes(b"not for this interpreter")
    with pytest.raises(ImportError, match="is not built"):
        bd._load_calls()
    shutil.copy(bd._calls.__file__, tmp_path)
    assert bd._load_calls().Call
