"""The binding's native marshalling (no GPU): every argument arrives in its place, and what is no device tensor is refused before
anything is called."""
import ctypes
import importlib.machinery
import inspect
import os

import numpy as np
import pytest
import torch

import paper_2511_16947_amd as fm

U = ctypes.c_uint64


class DeviceTensor:
    """What the marshalling asks of a tensor."""
    is_cuda = True

    def __init__(self, at, contiguous=True):
        self.at, self.contiguous = at, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.at

    def numel(self):
        return 5000


@pytest.fixture
def call():
    fm.load_library()
    return fm._call


def test_module_is_this_interpreters(call):
    """No other interpreter finds it: its name carries the tag."""
    path = os.path.join(os.path.dirname(fm.__file__), "_call" + importlib.machinery.EXTENSION_SUFFIXES[0])
    assert fm._call.__self__.__file__ == path == fm.CALL_PATH
    assert importlib.machinery.EXTENSION_SUFFIXES[0] != ".so"


@pytest.mark.parametrize("n", [0, 1, 3, 5, 6, 13, 22])
def test_arguments_arrive_in_order(call, n):
    seen = []
    fn = ctypes.CFUNCTYPE(ctypes.c_int, *[U] * (n + 2))(lambda *a: seen.append(a) or -7)
    kinds = "".join("ti"[i % 2] for i in range(n))
    args = [(DeviceTensor((1 << 63) + i) if i % 4 else None) if k == "t" else -i for i, k in enumerate(kinds)]
    want = [((1 << 63) + i if i % 4 else 0) if k == "t" else -i % (1 << 64) for i, k in enumerate(kinds)]
    assert call(ctypes.cast(fn, ctypes.c_void_p).value, kinds, lambda: 1234, 77, *args) == -7
    assert seen == [(77, *want, 1234)]


@pytest.mark.parametrize("kind,arg,error", [
    ("t", torch.zeros(4), AssertionError), ("t", DeviceTensor(8, False), AssertionError), ("t", 4096, AttributeError),
    ("t", "x", AttributeError), ("t", DeviceTensor(1.5), TypeError), ("i", None, TypeError), ("i", 1.0, TypeError),
    ("i", DeviceTensor(8), TypeError), ("i", torch.zeros(1), TypeError)])
def test_what_is_refused(call, kind, arg, error):
    with pytest.raises(error):      # (address 1 would be called; the stream is asked for only when all is accepted)
        call(1, "i" + kind, lambda: pytest.fail("accepted"), 77, 3, arg)


class Index:
    def __index__(self):
        return -3


class AsParameter:
    def __init__(self, value):
        self._as_parameter_ = value


@pytest.mark.parametrize("arg", [
    np.int32(-3), np.int64(-3), np.int8(-3), np.array(-3), torch.tensor(-3), torch.tensor(-3, dtype=torch.int32), Index(),
    ctypes.c_int32(-3), AsParameter(-3), AsParameter(AsParameter(np.int64(-3)))])
def test_integers_of_every_kind(call, arg):
    """What ctypes takes for an int32_t: out of NumPy and torch too."""
    seen = []
    fn = ctypes.CFUNCTYPE(ctypes.c_int, *[U] * 3)(lambda *a: seen.append(a) or 0)
    assert call(ctypes.cast(fn, ctypes.c_void_p).value, "i", lambda: 9, 77, arg) == 0
    assert seen == [(77, -3 % (1 << 64), 9)]


@pytest.mark.parametrize("arg", [np.float32(1), np.array([3]), torch.tensor(1.0), torch.tensor([1, 2]), ctypes.c_int64(1), ctypes.c_uint32(1),
                                 AsParameter(1.0), AsParameter(None), "x", None])
def test_refused_integers(call, arg):
    with pytest.raises(TypeError) as info:
        call(1, "ii", lambda: pytest.fail("accepted"), 77, 3, arg)
    assert isinstance(info.value, ctypes.ArgumentError)      # what ctypes raises
    loop = AsParameter(0)
    loop._as_parameter_ = loop
    with pytest.raises(RecursionError):
        call(1, "i", lambda: pytest.fail("accepted"), 77, loop)


def test_kinds_match_the_prototypes():
    lib = fm.load_library()
    for name, kinds in fm._KINDS.items():
        types = getattr(lib, name).argtypes[1:-1]
        assert len(types) == len(kinds), name
        host = {"fine_cayley_placement": (1, 3)}.get(name, ())      # addresses of host arrays
        for i, (t, k) in enumerate(zip(types, kinds)):
            assert (k == "t") == (t is ctypes.c_void_p and i not in host), (name, i)


@pytest.mark.parametrize("name", [n for n in fm._KINDS if n not in ("fine_cayley_placement",)])
def test_wrappers_refuse_host_tensors(name):
    shape = fm.Shape(256, 128, 256, 8, 2, 4, fm.FINE_F32)
    f = getattr(fm, name)
    params = list(inspect.signature(f).parameters)[1:]
    values = [1 if p in ("rank", "slots", "n", "seed", "alpha_num", "alpha_den", "ranks_per_node", "accumulate") else torch.zeros(300) for p in params]
    with pytest.raises(AssertionError):
        f(shape, *values)
