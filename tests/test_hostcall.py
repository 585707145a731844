"""The binding's call helper: what it passes for each kind of argument, and what it refuses."""
import ctypes as C
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest

from paper_2603_22910_amd import binding as ek
from paper_2603_22910_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", params=["_hostcall", "ctypes"])
def call(request):
    if not os.path.exists(ek.LIB_PATH):
        build.build_library()
    if request.param == "ctypes":
        return ek.call_by_ctypes
    if not os.path.exists(build.HOSTCALL_PATH) and build.build_hostcall() is None:
        pytest.skip("no C compiler or no Python.h")
    from paper_2603_22910_amd import _hostcall
    return _hostcall.call


def test_library_loads_without_the_helper():
    """Every entry point is there where the helper is not: the rest of the binding never needs it, a decode loop's calls go by ctypes."""
    code = ("import sys; sys.modules['paper_2603_22910_amd._hostcall'] = None\n"
            "from paper_2603_22910_amd import binding as ek\n"
            "print(ek.status_string(0))\n"
            "c = ek.LayerCache(1 << 20, 1 << 20, 512, 64, [0], [60], [64])\n"
            "try: ek.cache_append(ek.make_shape(8, 8, 64, 256, 'f32'), c, 1 << 20, 1 << 20, [5], stream=0)\n"
            "except ek.EchoKVError as e: print(e.code == ek.ERR_CAPACITY, ek._call is ek.call_by_ctypes)\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert out.returncode == 0, out.stderr
    assert out.stdout.split() == ["ok", "True", "True"]


def test_helper_is_built_for_one_python_and_not_a_need_of_the_build(monkeypatch, tmp_path, capsys):
    assert build.HOSTCALL_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(build, "HOSTCALL_PATH", str(tmp_path / "_hostcall.so"))
    for compiler in ("/bin/false", "/no/such/compiler"):
        monkeypatch.setattr(build.shutil, "which", lambda _: compiler)
        assert build.build_hostcall() is None
        assert "not built" in capsys.readouterr().err


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
