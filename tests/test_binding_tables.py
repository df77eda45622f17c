"""The binding's native marshalling against the per-element Python it stands for."""
import ctypes
import os
import subprocess
import sys
import types

import numpy as np
import pytest
import torch

mics = pytest.importorskip("paper_2205_00119_amd")


def address(x):
    if x is None:
        return None
    if isinstance(x, int):
        return x
    if not x.is_contiguous():
        raise ValueError("tensor must be contiguous")
    return x.data_ptr()


class Like:
    """Not a tensor, but answers like one."""

    def __init__(self, ptr, contiguous=True):
        self.ptr, self.contiguous = ptr, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.ptr


class Sub(torch.Tensor):
    pass


BASE = torch.zeros(6, 8)
ITEMS = {
    "tensors": [BASE, BASE[2], BASE[1, 3:], torch.empty(0), torch.zeros((), dtype=torch.bfloat16)],
    "parameters": (torch.nn.Parameter(torch.zeros(3)), torch.zeros(3).as_subclass(Sub)),
    "mixed": [None, 0, 4096, 2 ** 64 - 16, True, Like(4096), BASE[0]],
    "rows of a tensor": BASE,
    "none": [],
    "128": [BASE[i % 6] for i in range(128)],
}


@pytest.mark.parametrize("name", list(ITEMS))
def test_pointer_tables(name):
    items = ITEMS[name]
    got = mics._table(items)
    want = (ctypes.c_void_p * len(items))(*[address(x) for x in items])
    assert type(got) is type(want) and bytes(got) == bytes(want)
    for x in items:
        a, b = ctypes.c_void_p(mics._dev_ptr(x)).value, ctypes.c_void_p(address(x)).value
        assert a == b


@pytest.mark.parametrize("bad,error", [(BASE.t(), ValueError), (BASE[:, 1], ValueError), (Like(8, False), ValueError),
                                       ("text", AttributeError), (1.5, AttributeError)])
def test_what_is_no_address_is_refused(bad, error):
    for call in (lambda: mics._table([BASE, bad]), lambda: mics._dev_ptr(bad)):
        with pytest.raises(error):
            call()
    with pytest.raises(TypeError):
        mics._table(iter([BASE]))


@pytest.mark.parametrize("kind", ["csr", "mkldnn", "vmap"])
def test_tensors_without_an_address_raise_what_their_methods_raise(kind):
    def check(x):
        with pytest.raises(RuntimeError) as want:
            address(x)
        for call in (lambda: mics._table([BASE, x]), lambda: mics._dev_ptr(x)):
            with pytest.raises(RuntimeError) as got:
                call()
            assert type(got.value) is type(want.value) and str(got.value) == str(want.value)
        return BASE[0]

    if kind == "vmap":
        torch.func.vmap(check)(BASE)
    else:
        check(BASE.to_sparse_csr() if kind == "csr" else BASE.to_mkldnn())


@pytest.mark.parametrize("segs", [[], [(1, 2, 3, 4)], ((5, 0, 2 ** 40, 7), [8, 9, 10, 11]), [(1, 2)], [()],
                                  [tuple(np.int64(x) for x in (3, 4, 5, 6)), np.arange(4)], [(1.0, 2.9, True, "7")],
                                  [(-1, 2 ** 64 + 5, 0, 0)], np.arange(8).reshape(2, 4)])
def test_segment_arrays(segs):
    got = mics._segments(segs)
    want = (mics.mics_segment * len(segs))(*[mics.mics_segment(*map(int, sg)) for sg in segs])
    assert type(got) is type(want) and bytes(got) == bytes(want)


@pytest.mark.parametrize("segs,error", [([(1, 2, 3, 4, 5)], TypeError), ([7], TypeError), ([("x", 0, 0, 0)], ValueError)])
def test_what_is_no_segment_is_refused(segs, error):
    with pytest.raises(error):
        mics._segments(segs)


DROPPED = """
import ctypes
import paper_2205_00119_amd as mics

class Item:
    def __init__(self, outer):
        self.outer = outer
        outer.append(self)
    def __iter__(self):
        self.outer.clear()
        return iter((1, 2))
    def __length_hint__(self):
        return 2

outer = []
Item(outer)
assert bytes(mics._segments(outer)) == bytes((mics.mics_segment * 1)(mics.mics_segment(1, 2)))

class Address:
    def __init__(self, outer):
        self.outer = outer
        outer.append(self)
    def is_contiguous(self):
        self.outer.clear()
        return True
    def data_ptr(self):
        return 4096

Address(outer)
assert bytes(mics._table(outer)) == bytes((ctypes.c_void_p * 1)(4096))
"""


def test_an_item_that_leaves_its_list_while_it_is_read():
    """The list's reference is the item's last one.  The allocator overwrites freed objects, in a process of
    its own."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", DROPPED], cwd=root, env=dict(os.environ, PYTHONMALLOC="debug"),
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr


T = [torch.zeros(8) for _ in range(6)]
HYPER = dict(lr=0.5, beta1=0.25, beta2=0.125, eps=1e-3, weight_decay=0.75, step=7)
SEGS = [(5, 6, 7, 8), (1, 2), (2 ** 40, 0, -1, 3)]
CALLS = {
    "gather": ("hier_gather_reorder", (T[0], T[1:3], 11, 12, 4, 2, 2), {}),
    "gather_coalesced": ("hier_gather_reorder_coalesced", (T[0], (T[1], 4096), SEGS, 4, 2, 4), {}),
    "reduce": ("reduce_scatter_accum", (T[0], T, 3, 4, True), {}),
    "reduce_typed": ("reduce_scatter_accum_typed", (T[0], T[2:], 3, -1, 0, 2), {}),
    "reduce_coalesced": ("reduce_scatter_accum_coalesced", (None, T, tuple(SEGS), 5), {}),
    "reduce_coalesced_typed": ("reduce_scatter_accum_coalesced_typed", (T[0], [None, 16], [], False, 1), {}),
    "average": ("replica_average", (T[3], [T[1]] * 128, 9, 0.1), {}),
    "adam": ("adam_shard", (T[0], T[1], T[2], T[3], T[4], 21), HYPER),
    "adam_typed": ("adam_shard_typed", (T[0], T[1], T[2], None, 1, T[4], 2 ** 64 + 21), HYPER),
    "update": ("replica_average_adam_shard", (T[0], T[1], T[2], T[3], T[4:], 21, 1e300), HYPER),
    "update_typed": ("replica_average_adam_shard_typed", (T[0], T[1], T[2], T[3], 2 ** 32 + 1, T[4:], 21, 3e-42), HYPER),
}
LIKE = {"as it is": lambda x: x, "numpy's integers": lambda x: np.int64(x) if type(x) is int and abs(x) < 2 ** 40 else x,
        "whole numbers": lambda x: int(x) if type(x) is float and x < 1e6 else x,
        "tuples": lambda x: tuple(x) if type(x) is list else x, "parameters": lambda x: torch.nn.Parameter(x) if x is T[0] else x,
        "not contiguous": lambda x: BASE.t() if x is T[0] else x, "text": lambda x: "7" if type(x) is int else x,
        "too many": lambda x: x * 65 if type(x) is list and len(x) in (2, 3) else x}


@pytest.mark.parametrize("like", list(LIKE))
@pytest.mark.parametrize("call", list(CALLS))
def test_whole_calls_hand_over_what_ctypes_does(monkeypatch, call, like):
    """Both ways with the library's entry point replaced by one that records its arguments."""
    name, args, kwargs = CALLS[call]
    args, kwargs = [LIKE[like](x) for x in args], {k: LIKE[like](x) for k, x in kwargs.items()}
    real, seen = getattr(mics.lib, "mics_" + name), []

    def record(*got):
        got = list(got)
        ints = [x for x in args if isinstance(x, (list, tuple))]
        for i, kind in enumerate(real.argtypes):
            if kind is ctypes.POINTER(mics.mics_segment):
                got[i] = [tuple(getattr(got[i][t], f) for f, _ in mics.mics_segment._fields_) for t in range(len(ints[1]))]
            elif i == TABLE[name]:
                got[i] = list((ctypes.c_void_p * len(ints[0])).from_address(got[i]))
        seen.append(got)
        return 0

    stub = ctypes.CFUNCTYPE(ctypes.c_int, *real.argtypes)(record)
    entries = ["mics_" + n for n in ENTRIES]
    addresses = [ctypes.cast(getattr(mics.lib, n), ctypes.c_void_p).value for n in entries]
    at = entries.index("mics_" + name)
    fake = addresses[:at] + [ctypes.cast(stub, ctypes.c_void_p).value] + addresses[at + 1:]

    def outcome():
        try:
            return getattr(mics, "mics_" + name)(*args, stream=64, **kwargs), seen.pop()
        except Exception as e:                                      # noqa: BLE001
            return type(e), str(e)

    mics._marshal.bind(tuple(fake), mics._device, mics._raw_stream)
    monkeypatch.setattr(mics, "lib", types.SimpleNamespace(**{"mics_" + name: stub}))
    try:
        fast = outcome()
        asked = getattr(mics._marshal, call)
        monkeypatch.setattr(mics, "_marshal", types.SimpleNamespace(**{**vars(mics._marshal), call: lambda *a: None}))
        assert fast == outcome()
        if like == "as it is":
            positional = [*args, *[kwargs[k] for k in ("lr", "beta1", "beta2", "eps", "weight_decay", "step") if k in kwargs], 64]
            assert asked(*positional) == 0                          # this one does go past ctypes
    finally:
        monkeypatch.undo()
        mics._marshal.bind(tuple(addresses), mics._device, mics._raw_stream)


ENTRIES = ("hier_gather_reorder", "hier_gather_reorder_coalesced", "reduce_scatter_accum", "reduce_scatter_accum_typed",
           "reduce_scatter_accum_coalesced", "reduce_scatter_accum_coalesced_typed", "replica_average", "adam_shard",
           "adam_shard_typed", "replica_average_adam_shard", "replica_average_adam_shard_typed")
TABLE = dict(hier_gather_reorder=1, hier_gather_reorder_coalesced=1, reduce_scatter_accum=1, reduce_scatter_accum_typed=1,
             reduce_scatter_accum_coalesced=1, reduce_scatter_accum_coalesced_typed=1, replica_average=1, adam_shard=None,
             adam_shard_typed=None, replica_average_adam_shard=4, replica_average_adam_shard_typed=5)


def bound(device, raw_stream, entry=None):
    """Binds the entry points with other callables for the current stream, every entry point being `entry` if given."""
    addresses = [ctypes.cast(entry or getattr(mics.lib, "mics_" + n), ctypes.c_void_p).value for n in ENTRIES]
    mics._marshal.bind(tuple(addresses), device, raw_stream)


def positional(call, stream):
    args, kwargs = CALLS[call][1:]
    return [*args, *[kwargs[k] for k in ("lr", "beta1", "beta2", "eps", "weight_decay", "step") if k in kwargs], stream]


@pytest.mark.parametrize("where", ["device", "raw stream"])
@pytest.mark.parametrize("call", list(CALLS))
def test_an_interrupt_while_the_current_stream_is_asked_for(call, where):
    """Signals are handled in the Python code that names the current stream: what they raise leaves the call, nothing runs."""
    def interrupted(*_):
        raise KeyboardInterrupt("now")

    ran = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: ran.append(1) or 0)
    try:
        bound(interrupted if where == "device" else (lambda: 0), interrupted, entry)
        with pytest.raises(KeyboardInterrupt, match="now"):
            getattr(mics._marshal, call)(*positional(call, None))
        assert not ran
    finally:
        bound(mics._device, mics._raw_stream)


@pytest.mark.parametrize("k", [1, 3, 2 ** 32 + 2, 2 ** 64 + 2, 2 - 2 ** 32, 2 - 2 ** 64])
@pytest.mark.parametrize("call", ["gather", "gather_coalesced"])
def test_the_number_of_stage1_buffers_is_compared_as_it_is(call, k):
    """Two buffers and a k that is not 2, also one that is 2 in its low 32 or 64 bits."""
    name, args, _ = CALLS[call]
    at = 5 if call == "gather" else 4
    assert args[at] == 2
    wrong = [*args[:at], k, *args[at + 1:]]
    ran = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: ran.append(1) or 0)
    try:
        bound(mics._device, mics._raw_stream, entry)
        with pytest.raises(ValueError, match=f"expected k = {k} stage-1 buffers, got 2"):
            getattr(mics, "mics_" + name)(*wrong, stream=64)
        assert not ran
    finally:
        bound(mics._device, mics._raw_stream)


class Stream:
    def __init__(self, handle):
        self.handle = handle

    @property
    def cuda_stream(self):
        if isinstance(self.handle, BaseException):
            raise self.handle
        return self.handle


def as_array(segs):
    arr = (mics.mics_segment * len(segs))()
    for a, sg in zip(arr, segs):
        for (field, _), x in zip(mics.mics_segment._fields_, sg):
            setattr(a, field, x % 2 ** 64)
    return arr


def is_segments(x):
    return isinstance(x, (list, tuple)) and len(x) == len(SEGS) and all(a is b for a, b in zip(x, SEGS))


FORMS = {"a stream object": lambda x: Stream(x) if type(x) is int and x == 64 else x,
         "segments as lists": lambda x: [list(s) for s in x] if is_segments(x) else x,
         "an array of segments": lambda x: as_array(x) if is_segments(x) else x,
         "numpy's floats": lambda x: np.float64(x) if type(x) is float else x,
         "whole numbers": lambda x: int(x) if type(x) is float and x == int(x) and x < 1e6 else x}


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("call", list(CALLS))
def test_forms_of_arguments_that_go_past_ctypes(call, form):
    """What a call made without ctypes hands over does not depend on the form; the plain ones are compared with ctypes above."""
    name = CALLS[call][0]
    real, seen = getattr(mics.lib, "mics_" + name), []

    def record(*got):
        got = list(got)
        for i, kind in enumerate(real.argtypes):
            if kind is ctypes.POINTER(mics.mics_segment):
                got[i] = [tuple(getattr(got[i][t], f) for f, _ in mics.mics_segment._fields_) for t in range(got[i + 1])]
            elif i == TABLE[name]:
                got[i] = list((ctypes.c_void_p * len(CALLS[call][1][i])).from_address(got[i]))
        seen.append(got)
        return 0

    plain = [1.0 if type(x) is float and x == 1e300 else x for x in positional(call, 64)]
    if "weight_decay" in CALLS[call][2]:
        plain[-3] = 0.0                                             # a whole number among them
    stub = ctypes.CFUNCTYPE(ctypes.c_int, *real.argtypes)(record)
    try:
        bound(mics._device, mics._raw_stream, stub)
        for args in (plain, [FORMS[form](x) for x in plain]):
            assert getattr(mics._marshal, call)(*args) == 0
        assert seen[0] == seen[1]
    finally:
        bound(mics._device, mics._raw_stream)


def test_a_stream_object_that_raises_or_has_no_handle():
    ran = []
    entry = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: ran.append(1) or 0)
    try:
        bound(mics._device, mics._raw_stream, entry)
        for raised in (KeyboardInterrupt("now"), ZeroDivisionError("x")):
            with pytest.raises(type(raised)):
                mics.mics_replica_average(T[0], T[1:3], 4, 1.0, Stream(raised))
        with pytest.raises(AttributeError, match="cuda_stream"):
            mics.mics_replica_average(T[0], T[1:3], 4, 1.0, "7")
        assert mics._marshal.average(T[0], T[1:3], 4, 1.0, True) is None         # left to ctypes
        assert mics._marshal.average(T[0], T[1:3], 4, 1.0, Stream(None)) is None
        assert mics._marshal.reduce_coalesced(T[0], T, (ctypes.c_size_t * 4)(), True, 64) is None
        assert mics._marshal.average(T[0], T[1:3], 4, 10 ** 400, 64) is None
        assert not ran
    finally:
        bound(mics._device, mics._raw_stream)
