"""The Python binding by itself (no GPU): copies and pickles of a Shape, and the stream handle."""
import copy
import pickle
from dataclasses import dataclass

import pytest
import torch

import paper_2511_16947_amd as fm

ARGS = (256, 128, 256, 8, 2, 4, fm.FINE_F32, fm.FLAG_LOCALITY)


@dataclass(frozen=True)
class NamedShape(fm.Shape):
    name: str = "layer"

    @property
    def rows_per_rank(self):
        return self.P // self.G


@pytest.mark.parametrize("copy_of", [copy.copy, copy.deepcopy, lambda s: pickle.loads(pickle.dumps(s))])
def test_copies_keep_their_class(copy_of):
    for s in (fm.Shape(*ARGS), NamedShape(*ARGS, name="ffn.3")):
        fm.fine_workspace_bytes(s, fm.WS_FFN)      # with and without the converted form in place
        for t in (copy_of(s), copy_of(copy_of(s))):
            assert type(t) is type(s) and t == s
            assert fm.fine_workspace_bytes(t, fm.WS_FFN) == fm.fine_workspace_bytes(s, fm.WS_FFN) > 0
    assert t.name == "ffn.3" and t.rows_per_rank == 128


def test_pickle_of_the_fields_alone():
    """What a dataclass without methods for pickling writes: the class and its fields."""
    s = object.__new__(fm.Shape)
    s.__dict__.update(zip(("T", "d", "f", "E", "K", "G", "dtype", "flags"), ARGS))
    assert s == fm.Shape(*ARGS)
    assert fm.fine_workspace_bytes(s, fm.WS_SCHED) == fm.fine_workspace_bytes(fm.Shape(*ARGS), fm.WS_SCHED)


def test_shapes_that_no_call_can_take_can_be_made():
    assert fm.Shape(2.5, *ARGS[1:]).P == 5.0
    with pytest.raises(TypeError):
        fm.fine_workspace_bytes(fm.Shape(2.5, *ARGS[1:]), fm.WS_FFN)


class TestStream:
    """The stream handle comes from torch.cuda.current_stream() wherever the shorter way is not the same."""

    class Stream:
        cuda_stream = 1234

    @pytest.fixture(autouse=True)
    def functions(self, monkeypatch):
        monkeypatch.setattr(torch._C, "_cuda_isInBadFork", lambda: False, raising=False)
        monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device, raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream", lambda: self.Stream)

    @pytest.mark.parametrize("name", ["_cuda_isInBadFork", "_cuda_getCurrentRawStream", "_cuda_getDevice"])
    def test_without_the_functions(self, monkeypatch, name):
        monkeypatch.delattr(torch._C, name)
        assert fm._stream() == 1234

    def test_with_them(self):
        assert fm._stream() == 103

    def test_in_a_forked_child(self, monkeypatch):
        """Forked after the GPU was initialised: torch decides (it refuses)."""
        monkeypatch.setattr(torch._C, "_cuda_isInBadFork", lambda: True)
        assert fm._stream() == 1234
