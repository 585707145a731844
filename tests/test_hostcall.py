"""The binding's call helper: what it passes for each kind of argument, and what it refuses."""
import ctypes as C

import numpy as np
import pytest

from paper_2603_22910_amd import binding as ek


@pytest.fixture(scope="module")
def call():
    ek.load()
    return ek._call


@pytest.mark.parametrize("n", range(1, 15))
def test_arguments_arrive_in_their_places(call, n):
    seen = []
    kinds = [C.c_void_p, C.c_int64]
    fn = C.CFUNCTYPE(C.c_int, *(kinds[i % 2] for i in range(n)))(lambda *a: seen.extend(a) or n - 3)
    arr = np.arange(4, dtype=np.int32)
    args = [(None, 7, arr, -(1 << 40))[i % 4] for i in range(n)]
    assert call(C.cast(fn, C.c_void_p).value, *args) == n - 3
    assert seen == [(None, 7, arr.ctypes.data, -(1 << 40))[i % 4] for i in range(n)]


def test_structures_go_by_address_and_others_are_refused(call):
    sh = ek.make_shape(8, 8, 64, 256, "f32")
    fn = C.CFUNCTYPE(C.c_int, C.POINTER(ek.Shape))(lambda p: p.contents.n_retained)
    at = C.cast(fn, C.c_void_p).value
    assert call(at, sh) == 256
    for bad, err in ((1.5, TypeError), ("x", TypeError), (np.zeros((4, 4))[:, 1], ValueError), (object(), TypeError)):
        with pytest.raises((err, BufferError)):
            call(at, bad)
    for bad in ((at,), (at, *range(15))):
        with pytest.raises(TypeError):
            call(*bad)
    with pytest.raises(ValueError):
        call(0, 1)
    with pytest.raises(TypeError):                    # a shape has to be a Shape
        ek.cache_append(np.zeros(32, np.uint8), ek.LayerCache(1 << 20, 1 << 20, 512, 64, [0], [0], [64]), 1, 1, [1], stream=0)
