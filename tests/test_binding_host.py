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


def zero_stride_views():
    """[4, 3, 8] logits of which one dimension repeats the same memory."""
    return {"sequences": torch.zeros(1, 3, 8).expand(4, 3, 8), "positions": torch.zeros(4, 1, 8).expand(4, 3, 8),
            "both": torch.zeros(8).expand(4, 3, 8)}


@pytest.mark.parametrize("form", ["sequences", "positions", "both"])
def test_rows_that_repeat_the_same_memory_are_refused(library, form):
    """A stride of 0 means dense rows to the library, which would then read past the end of an expanded tensor."""
    lib = library()
    x = dev(zero_stride_views()[form])
    row, draft = torch.zeros(4, dtype=torch.int32), torch.zeros(4, 2, dtype=torch.int32)
    ids, val = dev(torch.zeros(4, 5, dtype=torch.int32)), dev(torch.zeros(4, 5))
    for call in (lambda: binding.verify_block(x, x, x, draft, torch.zeros(4, 3), workspace=dev(torch.zeros(256))),
                 lambda: binding.cloud_topk(x, x, row, topk=5),
                 lambda: binding.edge_resample(ids, val, x, row, torch.zeros(4))):
        with pytest.raises(ValueError, match="same memory"):
            call()
    rows = dev(torch.zeros(8).expand(4, 8))
    for call in (lambda: binding.steer_rows(rows, rows, rows, torch.zeros(4)),
                 lambda: binding.sample_rows(rows, torch.zeros(4))):
        with pytest.raises(ValueError, match="same memory"):
            call()
    assert not any(name.startswith(("specsteer_verify", "specsteer_cloud", "specsteer_edge")) for name, _ in lib.calls)


def test_a_zero_stride_of_a_dimension_of_one_is_no_repetition(library):
    """Nothing is repeated along a dimension of one: its stride means nothing and is passed on as dense."""
    lib = library()
    one = dev(torch.zeros(8).as_strided((1, 1, 8), (0, 0, 1)))
    row = torch.zeros(1, dtype=torch.int32)
    binding.cloud_topk(one, one, row, topk=5)
    binding.edge_resample(dev(torch.zeros(1, 5, dtype=torch.int32)), dev(torch.zeros(1, 5)), one, row, torch.zeros(1))
    binding.sample_rows(dev(torch.zeros(8).as_strided((1, 8), (0, 1))), torch.zeros(1))
    assert [n for n, _ in lib.calls] == ["specsteer_cloud_topk", "specsteer_edge_resample", "specsteer_workspace_bytes",
                                         "specsteer_verify_block"]


@pytest.mark.parametrize("device", ["cpu", "meta"])
@pytest.mark.parametrize("entry", ["verify_block_raw", "verify_block_static_raw"])
def test_raw_entry_points_refuse_host_tensors(monkeypatch, device, entry):
    """They check nothing else, but the stream they look up by themselves is that of the logits' device: logits on no
    GPU end there, on a machine that has one too, before the kernel is handed a host address."""
    lib = Recorder()
    monkeypatch.setattr(binding, "library", lambda: lib)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 0, raising=False)
    x = torch.zeros(1, 2, 8, device=device)
    p = binding.make_params(1, 1, 8, torch.float32, lam=0.5, beta=1.0, temperature=1.0)
    out = [torch.zeros(1, dtype=torch.int32), torch.zeros(1, dtype=torch.int32), torch.zeros(1), None, None]
    extra = [torch.zeros(256)] if entry == "verify_block_raw" else []
    with pytest.raises(ValueError, match="device"):
        getattr(binding, entry)(x, x, x, torch.zeros(1, 1, dtype=torch.int32), None, torch.zeros(1, 2), p, *out, *extra)
    assert lib.calls == []
