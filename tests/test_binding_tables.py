"""The binding's native marshalling against the per-element Python it stands for."""
import ctypes
import os
import subprocess
import sys

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
