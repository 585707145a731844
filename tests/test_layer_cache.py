"""The C view of a LayerCache follows its tensors and arrays: replaced storage, tensors and arrays assigned anew (a freed object's id comes
back), width and pool size."""
import numpy as np
import pytest
import torch

from paper_2603_22910_amd import binding as ek


def cache(rows=8):
    return ek.LayerCache(torch.zeros(rows, 4), torch.zeros(rows, 4), 4, rows, [0], [1], [rows])


def pointers(c):
    s = c.as_c()
    return [s.k, s.v] + [np.ctypeslib.as_array(p, (1,)).ctypes.data for p in (s.seq_start, s.seq_len, s.seq_cap)]


def expected(c):
    return [c.k.data_ptr(), c.v.data_ptr(), c.seq_start.ctypes.data, c.seq_len.ctypes.data, c.seq_cap.ctypes.data]


@pytest.mark.parametrize("name", ["k", "v"])
def test_replaced_storage(name):
    c = cache()
    assert pointers(c) == expected(c)
    getattr(c, name).data = torch.zeros(4096, 4)
    assert pointers(c) == expected(c)


@pytest.mark.parametrize("name", ["k", "v", "seq_start", "seq_len", "seq_cap"])
def test_two_assignments_between_calls(name):
    for rows in range(16, 56, 2):                  # a pool grown twice: the second object often sits where the first one sat
        c = cache()
        assert pointers(c) == expected(c)
        kept = []                                  # the memory stays in use, the objects go
        for n in (rows, rows + 1):
            if name in "kv":
                kept.append(getattr(c, name).data)
            setattr(c, name, None)
            setattr(c, name, torch.zeros(n, 4) if name in "kv" else np.ones(1, np.int64 if name == "seq_start" else np.int32))
        assert pointers(c) == expected(c)


def test_nothing_changed_is_the_same_view():
    c = cache()
    assert c.as_c() is c.as_c()
    c.width = 2
    assert c.as_c().width == 2
    c.pool_tokens = 4
    assert c.as_c().pool_tokens == 4
    assert ek.LayerCache(None, None, 0, 8, [0], [0], [8]).as_c().k is None
