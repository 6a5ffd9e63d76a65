"""The binding's native wrappers against its general path: what they take they answer alike, everything else they leave to it, and
without them it answers everything."""
import os
import shutil
import subprocess
import warnings

import pytest
import torch

from paper_2603_16219_amd import binding
from paper_2603_16219_amd import build as binding_build


@pytest.fixture(scope="module", autouse=True)
def loaded():
    binding.library()
    assert binding._calls is not None


def test_host_tensors_and_other_objects_are_left_to_the_general_path():
    """Which refuses or converts them (CPU)."""
    x, i, u = torch.zeros(2, 3, 8), torch.zeros(2, dtype=torch.int32), torch.zeros(2)
    c = binding._calls
    for g in (x, x.bfloat16(), x.double(), torch.zeros(2, 3, 8, device="meta"), None, 1, x.numpy()):
        assert c.verify_block(g, g, g, torch.zeros(2, 2, dtype=torch.int32), torch.zeros(2, 3), 0.5, 1.0, 1.0, None, False, False, None,
                              False, False) is None
        assert c.steer_rows(g, g, g, u, 1.0, 1.0, False, False) is None
        assert c.cloud_topk(g, g, i, 1.0, 4) is None
        assert c.edge_resample(i.view(2, 1), u.view(2, 1), g, i, u, 1.0, 1.0, False) is None
    assert c.steer_rows() is None and c.cloud_topk(x) is None  # another number of arguments
    with pytest.raises(ValueError, match="device"):
        binding.steer_rows(x[:, 0], x[:, 0], x[:, 0], u)


@pytest.fixture
def not_loaded(monkeypatch):
    """The binding as it is before its first call; as it was afterwards."""
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_calls", None)
    return monkeypatch


def loads_without_wrappers(because):
    p = binding.make_params(2, 3, 1000, torch.float32, lam=0.5, beta=1.0, temperature=1.0)
    with pytest.warns(RuntimeWarning, match=because):
        assert binding.version() >= 100
    assert binding._lib is not None and binding._calls is None
    with warnings.catch_warnings():
        warnings.simplefilter("error")  # one warning, not one a call
        assert binding.first_window(p) == 3 and binding.workspace_bytes(p) > 0


@pytest.mark.parametrize("compiler", ["/nonexistent/g++", "false"])
def test_the_library_loads_where_the_wrappers_cannot_be_built(not_loaded, tmp_path, compiler):
    not_loaded.setattr(binding_build, "calls_path", lambda: str(tmp_path / "_calls.so"))
    not_loaded.setenv("CXX", compiler)
    loads_without_wrappers("not available")
    assert os.listdir(tmp_path) == []


def test_the_library_loads_where_the_wrappers_do_not(not_loaded, tmp_path):
    (tmp_path / "_calls.so").write_bytes(b"no shared object")
    not_loaded.setattr(binding_build, "calls_path", lambda: str(tmp_path / "_calls.so"))
    loads_without_wrappers("_calls.so")


def test_a_library_from_before_the_wrappers_loads(not_loaded, tmp_path):
    names = ("workspace_bytes", "verify_block", "verify_block_timed", "verify_block_static", "cloud_topk", "edge_resample")
    src = "".join(f"int specsteer_{n}(void) {{ return 1; }}\n" for n in names)
    src += "int specsteer_first_window(void) { return 3; }\nint specsteer_version(void) { return 100; }\nconst char *specsteer_status_string(int s) { return s ? \"\" : 0; }\n"
    (tmp_path / "old.c").write_text(src)
    old = str(tmp_path / "old.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", old, str(tmp_path / "old.c")], check=True)
    not_loaded.setattr(binding_build, "LIBRARY", old)
    loads_without_wrappers("specsteer_verify_block_unbound")


def test_wrappers_of_another_torch_or_other_sources_are_not_loaded(monkeypatch, tmp_path):
    """Their file's name says what they were built against."""
    here = binding_build.calls_path()
    assert os.path.exists(here) and binding_build.calls_path() == here
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "2.99.0")
        assert binding_build.calls_path() != here
    for i in range(len(binding_build.CALLS_SOURCES)):
        copies = [shutil.copy(p, tmp_path / os.path.basename(p)) for p in binding_build.CALLS_SOURCES]
        monkeypatch.setattr(binding_build, "CALLS_SOURCES", copies)
        assert binding_build.calls_path() == here
        with open(copies[i], "a") as f:
            f.write("\n")
        assert binding_build.calls_path() != here
        monkeypatch.undo()


def logits(dtype, B, k1, V, pad, odd):
    """Three tensors of one form: rows padded to a stride, and bases moved by an element."""
    gen = torch.Generator("cuda").manual_seed(B * V + pad)
    out = []
    for _ in range(3):
        flat = torch.randn(B * k1 * (V + pad) + odd, generator=gen, device="cuda").to(dtype)
        out.append(flat[odd:].view(B, k1, V + pad)[:, :, :V])
    return out


def both(monkeypatch, call):
    """The call by the native wrapper, which has to take it, and by the general path."""
    taken = []

    class Spy:
        def __getattr__(self, name):
            f = getattr(calls, name)

            def run(*a):
                out = f(*a)
                taken.append(out is not None)
                return out

            return run

    calls = binding._calls
    monkeypatch.setattr(binding, "_calls", Spy())
    native = call()
    assert taken == [True]
    monkeypatch.setattr(binding, "_calls", None)
    general = call()
    monkeypatch.setattr(binding, "_calls", calls)
    return native, general


def assert_alike(native, general):
    native, general = (x if isinstance(x, dict) else dict(enumerate(x)) for x in (native, general))
    assert list(native) == list(general)
    for k, a in native.items():
        b = general[k]
        if b is None:
            assert a is None, k
            continue
        assert type(a) is type(b) and a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and a.device == b.device, k
        assert not a.requires_grad and torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)), k


FORMS = [(1, 1, 40, 0, 0), (1, 5, 2049, 0, 0), (3, 3, 5001, 7, 1), (40, 2, 33000, 0, 0), (130, 4, 777, 1, 0), (64, 1, 151936, 0, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,k1,V,pad,odd", FORMS)
@pytest.mark.parametrize("greedy", [False, True])
def test_native_wrappers_answer_as_the_general_path(monkeypatch, dtype, B, k1, V, pad, odd, greedy):
    G, P, M = logits(dtype, B, k1, V, pad, odd)
    if B == 3:
        G, P, M = (torch.nn.Parameter(x) for x in (G, P, M))
    gen = torch.Generator("cuda").manual_seed(1)
    draft = torch.randint(0, V, (B, k1 - 1), generator=gen, device="cuda", dtype=torch.int32)
    lens = torch.randint(0, k1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    u = torch.rand(B, k1, generator=gen, device="cuda")
    row = torch.randint(0, k1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    ue = torch.rand(B, generator=gen, device="cuda")
    p = binding.make_params(B, k1 - 1, V, dtype, lam=0.5, beta=0.8, temperature=0.9)
    for kw in (dict(), dict(draft_len=lens, want_recovery_logprobs=True, want_draft_logprobs=True), dict(full_rows=True, beta=0),
               dict(workspace=torch.empty(binding.workspace_bytes(p) + 256, dtype=torch.uint8, device="cuda"))):
        out = both(monkeypatch, lambda: binding.verify_block(G, P, M, draft, u, **{**dict(lam=0.5, beta=0.8, temperature=0.9, greedy=greedy), **kw}))
        assert torch.all(out[0]["accepted_len"] >= 0)
        assert_alike(*out)
    rows = [x.detach()[:, 0] for x in (G, P, M)]
    assert_alike(*both(monkeypatch, lambda: binding.steer_rows(*rows, ue, beta=0.8, temperature=0.9, greedy=greedy, want_logprobs=B != 64)))
    assert_alike(*both(monkeypatch, lambda: binding.sample_rows(rows[0], ue.view(1, B), temperature=1, greedy=greedy)))
    top = both(monkeypatch, lambda: binding.cloud_topk(G, M, row, beta=0.8, topk=min(V, 33)))
    assert_alike(*top)
    idx, val = top[0]
    assert_alike(*both(monkeypatch, lambda: binding.edge_resample(idx, val, P, row, None if greedy else ue, beta=0.8, temperature=0.9, greedy=greedy)))


@pytest.mark.gpu
def test_what_has_to_be_converted_or_refused_goes_the_general_path(monkeypatch):
    B, k1, V = 4, 3, 500
    G, P, M = logits(torch.float32, B, k1, V, 0, 0)
    draft, u = torch.zeros(B, k1 - 1, dtype=torch.int32, device="cuda"), torch.rand(B, k1, device="cuda")
    row, ue = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.rand(B, device="cuda")
    idx, val = binding.cloud_topk(G, M, row, topk=8)
    c = binding._calls
    vb = lambda **kw: [kw.get(k, d) for k, d in dict(G=G, P=P, M=M, draft=draft, u=u, lam=0.5, beta=1.0, T=1.0, lens=None, rec=False, dlp=False, ws=None,
                                                     greedy=False, full=False).items()]
    assert c.verify_block(*vb()) is not None
    twice = G[:1].expand(B, k1, V)
    for kw in (dict(draft=draft.long()), dict(draft=draft.cpu()), dict(draft=draft[:, :1]), dict(u=u.double()), dict(u=u.t().contiguous().t()),
               dict(u=u[:, :2]), dict(G=G.bfloat16()), dict(G=G.transpose(1, 2).contiguous().transpose(1, 2)), dict(P=P[:, :2]),
               dict(G=twice, P=twice, M=twice), dict(lens=row.long()), dict(lens=row[:2]), dict(ws=torch.empty(1 << 20, dtype=torch.uint8)),
               dict(lam=torch.tensor(0.5)), dict(greedy=1), dict(G=G.half(), P=P.half(), M=M.half())):
        assert c.verify_block(*vb(**kw)) is None, kw.keys()
    g = G[:, 0]
    for args in ((g, g, g, u[:, 0], 1.0, 1.0, False, False), (g, g, g, ue.cpu(), 1.0, 1.0, False, False), (g, g, g, ue[:2], 1.0, 1.0, False, False),
                 (g, g, M[:, 0].contiguous(), ue, 1.0, 1.0, False, False)):
        assert c.steer_rows(*args) is None
    for args in ((G, M, row.long(), 1.0, 8), (G, M, row, 1.0, 0), (G, M, row, 1.0, 65), (G, M, row, 1.0, 8.0), (G, M, row[:2], 1.0, 8)):
        assert c.cloud_topk(*args) is None
    for args in ((idx[:, :4], val[:, :4], P, row, ue, 1.0, 1.0, False), (idx.long(), val, P, row, ue, 1.0, 1.0, False), (idx, val, P, row, None, 1.0, 1.0, False),
                 (idx, val[:, :4].contiguous(), P, row, ue, 1.0, 1.0, False), (idx, val, P, row, ue.double(), 1.0, 1.0, False)):
        assert c.edge_resample(*args) is None
    # converted there: the same answers as from what is ready
    want = binding.verify_block(G, P, M, draft, u, draft_len=row)
    got = binding.verify_block(G, P, M, draft.long().cpu(), u.double().t().contiguous().t(), draft_len=row.cpu().long())
    assert all(torch.equal(want[k], got[k]) for k in ("accepted_len", "next_token", "next_token_logprob"))
    # the library's own refusals: the same status either way
    for call in (lambda: binding.verify_block(G, P, M, draft, u, temperature=-1.0), lambda: binding.steer_rows(g, g, g, ue, temperature=0.0),
                 lambda: binding.verify_block(G, P, M, draft, u, workspace=torch.empty(256, dtype=torch.uint8, device="cuda")),
                 lambda: binding.edge_resample(idx, val, P, row, ue, temperature=float("inf"))):
        seen = []
        for calls in (c, None):
            monkeypatch.setattr(binding, "_calls", calls)
            with pytest.raises(binding.SpecSteerError) as e:
                call()
            seen.append((e.value.status, str(e.value)))
        monkeypatch.setattr(binding, "_calls", c)
        assert seen[0] == seen[1]
