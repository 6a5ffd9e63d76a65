"""What the Python binding hands to the library (CPU): the wrappers run on host tensors that claim to be on a device,
and a stand-in for the library looks at the pointers it is given instead of launching anything."""
import ctypes
import weakref

import pytest
import torch

from paper_2603_16219_amd import binding


class OnDevice(torch.Tensor):
    """A host tensor that passes for a device tensor; whatever is made from it does too."""

    @property
    def is_cuda(self):
        return True


def dev(t):
    return t.as_subclass(OnDevice)


class Recorder:
    """Takes the place of the library: `calls` holds the name and the arguments of every call, `look` may read the
    memory behind them while the call lasts."""

    def __init__(self, look=None):
        self.calls, self.look = [], look

    def __getattr__(self, name):
        def call(*args):
            self.calls.append((name, args))
            return self.look(args) if self.look else 0

        return call


@pytest.fixture
def library(monkeypatch):
    def install(look=None):
        lib = Recorder(look)
        monkeypatch.setattr(binding, "library", lambda: lib)
        monkeypatch.setattr(binding, "_stream", lambda device: 0)
        return lib

    return install


@pytest.mark.parametrize("layout", ["columns", "transposed", "dense"])
def test_edge_resample_hands_over_the_payload_it_was_given(library, monkeypatch, layout):
    """A payload that has to be copied first (columns of a wider one, a transposed one): both copies are alive, at
    addresses of their own, while the library reads them."""
    B, k = 3, 16
    index = torch.arange(B * 2 * k, dtype=torch.int32).reshape(B, 2 * k)
    value = -torch.arange(B * 2 * k, dtype=torch.float32).reshape(B, 2 * k)
    if layout == "columns":
        index, value = index[:, :k], value[:, :k]
    elif layout == "transposed":
        index, value = (t[:, :k].contiguous().t().contiguous().t() for t in (index, value))
    else:
        index, value = index[:, :k].contiguous(), value[:, :k].contiguous()
    want_i, want_v = index.clone().contiguous(), value.clone().contiguous()

    # the copies the wrapper makes: one that is gone when the library is called was freed too early
    made = []
    contiguous = torch.Tensor.contiguous

    def tracked(self, *a, **kw):
        out = contiguous(self, *a, **kw)
        if out is not self:
            made.append(weakref.ref(out))
        return out

    monkeypatch.setattr(OnDevice, "contiguous", tracked)
    seen = {}

    def look(args):
        seen["copies"], seen["dead"] = len(made), sum(r() is None for r in made)
        if not seen["dead"]:
            seen["index"] = (ctypes.c_int32 * (B * k)).from_address(args[0])[:]
            seen["value"] = (ctypes.c_float * (B * k)).from_address(args[1])[:]
        return 0

    library(look)
    S = dev(torch.zeros(B, 2, 64))
    binding.edge_resample(dev(index), dev(value), S, torch.zeros(B, dtype=torch.int32), torch.zeros(B))
    assert seen["copies"] == (0 if layout == "dense" else 2) and seen["dead"] == 0
    assert seen["index"] == want_i.reshape(-1).tolist() and seen["value"] == want_v.reshape(-1).tolist()
