"""GPU tests of single kernels at the sizes where their tiling can go wrong, against the float64 oracle.
Tolerances are those of tests/parity.py (1e-5 on a log-prob, tokens and lengths exact outside the 1e-6 bands)."""
import dataclasses

import pytest
import torch

import parity
from paper_2603_16219_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    from paper_2603_16219_amd import binding as b

    assert torch.cuda.is_available(), "GPU tests need a device"
    b.library()
    return b


def recipe(name, dtype, **size):
    return dataclasses.replace(W.scaled(W.WORKLOADS[name], name=f"{name}-{dtype}-{size}", **size), dtype=dtype)


def in_stages(binding, inp, *, lam, beta, temperature, draft_len=None, greedy=False):
    """The block by the timed call, which is a row pass and a recovery also for small blocks that the others take in one launch:
    what is said below about those two kernels holds of it at every size."""
    batch, k_max = inp["draft"].shape
    p = binding.make_params(batch, k_max, inp["G"].shape[2], inp["G"].dtype, lam=lam, beta=beta, temperature=temperature,
                            stride_b=inp["G"].stride(0), stride_t=inp["G"].stride(1), flags=binding.SS_FLAG_GREEDY if greedy else 0)
    ws = torch.empty(max(256, binding.workspace_bytes(p)), dtype=torch.uint8, device="cuda")
    out = {"accepted_len": torch.empty(batch, dtype=torch.int32, device="cuda"), "next_token": torch.empty(batch, dtype=torch.int32, device="cuda"),
           "next_token_logprob": torch.empty(batch, device="cuda"), "recovery_logprobs": None,
           "draft_logprobs": torch.empty(batch, k_max, 2, device="cuda")}
    binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"] if k_max else None, draft_len, inp["uniforms"], p,
                             *out.values(), ws, timed=True)
    return out


# Short log-prob rows are written by the recovery launch (5 sequences: up to 256 KiB a row, 26214 bf16 or 16384 fp32 logits),
# longer ones by a launch of their own, cut into segments of 512 vectors (4096 bf16 or 2048 fp32 logits): whole segments,
# one logit more and less, a last segment that holds only the logits past the last vector, less than a vector.
@pytest.mark.parametrize("beta", [0.0, 0.8])
@pytest.mark.parametrize("dtype,vocab", [("bf16", 4096), ("bf16", 4097), ("bf16", 8191), ("bf16", 3), ("f32", 2048),
                                         ("f32", 2049), ("f32", 6143), ("f32", 3),
                                         ("bf16", 26214), ("bf16", 26215), ("bf16", 28671), ("bf16", 28672), ("bf16", 28673),
                                         ("f32", 16384), ("f32", 16385), ("f32", 18431), ("f32", 18432), ("f32", 18433)])
def test_logprob_rows_at_segment_edges(binding, oracle, dtype, vocab, beta):
    w = recipe("c4", dtype, batch=5, k_max=3, vocab=vocab)
    inp = W.generate(w, "cuda")
    inp["draft_len"] = torch.tensor([3, 0, 4, 1, 2], dtype=torch.int32, device="cuda")  # 4 > k_max: flagged
    p = binding.make_params(5, 3, vocab, inp["G"].dtype, lam=w.lam, beta=beta, temperature=w.temperature)
    ws = torch.empty(binding.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    out = {"accepted_len": torch.empty(5, dtype=torch.int32, device="cuda"),
           "next_token": torch.empty(5, dtype=torch.int32, device="cuda"),
           "next_token_logprob": torch.empty(5, device="cuda"),
           "recovery_logprobs": torch.full((5, vocab), 7.0, device="cuda"),
           "draft_logprobs": None}
    binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["draft_len"], inp["uniforms"], p,
                             out["accepted_len"], out["next_token"], out["next_token_logprob"],
                             out["recovery_logprobs"], None, ws)
    torch.cuda.synchronize()
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])
    assert out["accepted_len"][2].item() == -1 and torch.all(out["recovery_logprobs"][2] == 7.0)  # left unwritten


# Log-prob rows of a recovery row in several parts: the parts only deliver, and one launch draws and writes the rows.
@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0), (True, 0.0)])
@pytest.mark.parametrize("dtype,batch,vocab", [("bf16", 4, 20 * 2048 + 5), ("bf16", 40, 75 * 2048 - 1), ("f32", 3, 65 * 1024),
                                               ("f32", 7, 260 * 1024 + 1)])
def test_logprob_rows_beside_the_draw(binding, oracle, dtype, batch, vocab, greedy, beta):
    w = recipe("c4", dtype, batch=batch, k_max=3, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=16)
    inp["draft_len"] = torch.tensor([i % 4 for i in range(batch)], dtype=torch.int32, device="cuda")
    inp["draft_len"][1] = 4  # flagged
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=beta,
                               temperature=w.temperature, draft_len=inp["draft_len"], greedy=greedy, want_recovery_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])
    assert out["accepted_len"][1].item() == -1


# fp32 rows without a draft, their log-probs written over the generalist's or a specialist's logits: the token is drawn first, whether
# the rows come from the recovery launch (16384) or later.
@pytest.mark.parametrize("over", ["G", "S_ctx", "S_noctx"])
@pytest.mark.parametrize("batch,vocab,beta", [(5, 16384, 0.8), (8, 70000, 0.8), (100, 200001, 0.8), (8, 200001, 0.0)])
def test_logprob_rows_in_place(binding, batch, vocab, beta, over):
    gen = torch.Generator("cuda").manual_seed(batch)
    rows = {k: torch.randn(batch, 1, vocab, generator=gen, device="cuda") for k in ("G", "S_ctx", "S_noctx")}
    u = torch.rand(batch, 1, generator=gen, device="cuda")
    none = torch.empty(batch, 0, dtype=torch.int32, device="cuda")
    want = binding.verify_block(*rows.values(), none, u, beta=beta, want_recovery_logprobs=True)
    p = binding.make_params(batch, 0, vocab, torch.float32, lam=0.5, beta=beta, temperature=1.0)
    ws = torch.empty(binding.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    out = {k: torch.empty_like(want[k]) for k in ("accepted_len", "next_token", "next_token_logprob")}
    binding.verify_block_raw(*rows.values(), None, None, u, p, *out.values(), rows[over], None, ws)
    assert torch.equal(out["next_token"], want["next_token"]) and torch.equal(out["accepted_len"], want["accepted_len"])
    assert torch.allclose(out["next_token_logprob"], want["next_token_logprob"], rtol=0, atol=2e-6)
    assert torch.allclose(rows[over][:, 0], want["recovery_logprobs"], rtol=0, atol=4e-6)


# The recovery launch: 4-wave workgroups of one chunk a wave while batch x chunks <= 8 x 256 (a single workgroup of 16 waves
# for 5 .. 8 chunks), then 16-wave parts, no more than rounds of 16 chunks, up to 128 sequences, then one workgroup of 16 waves
# per sequence up to 256 and of 8 beyond.  A chunk is 256 vectors (2048 bf16, 1024 fp32 logits), the logits past the last vector
# are a chunk of their own.
@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0), (True, 0.0)])
@pytest.mark.parametrize("dtype,batch,vocab", [
    ("bf16", 1, 4 * 2048), ("bf16", 1, 4 * 2048 + 1), ("bf16", 3, 7 * 2048 + 9), ("f32", 2, 4 * 1024 + 1), ("f32", 5, 3),
    ("bf16", 128, 16 * 2048), ("bf16", 128, 16 * 2048 + 5), ("f32", 100, 40 * 1024 + 3),
    ("bf16", 129, 4100), ("bf16", 257, 4100)])
def test_recovery_launch_shapes(binding, oracle, dtype, batch, vocab, greedy, beta):
    w = recipe("c4", dtype, batch=batch, k_max=1, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=64)
    inp["draft_len"] = torch.randint(0, 2, (batch,), generator=torch.Generator("cuda").manual_seed(batch), device="cuda",
                                     dtype=torch.int32)
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam,
                               beta=beta, temperature=w.temperature, draft_len=inp["draft_len"], greedy=greedy,
                               want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy,
                            want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])
    parity.compare(in_stages(binding, inp, lam=w.lam, beta=beta, temperature=w.temperature, draft_len=inp["draft_len"], greedy=greedy), ora,
                   inp["uniforms"], inp["draft_len"])


# Up to 128 rows without a draft: one launch while a 16-wave workgroup takes its row fast enough, with pairs of chunks where there is no
# steering term, else a launch for the chunk masses, four chunks a workgroup, and one for the draw.  Whole chunks and
# workgroups, pairs with and without a chunk over, whose second chunk is partial (one vector, a third, a half), one logit more, odd
# rows, a row that has a length (flagged).
@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0), (True, 0.0)])
@pytest.mark.parametrize("dtype,batch,vocab", [("bf16", 1, 20 * 2048), ("bf16", 3, 16 * 2048 + 1), ("bf16", 128, 17 * 2048 + 9),
                                               ("bf16", 4, 32 * 2048), ("bf16", 9, 76 * 2048), ("bf16", 9, 77 * 2048 - 3),
                                               ("f32", 9, 104 * 1024 + 1), ("bf16", 9, 33 * 2048 + 1),
                                               ("f32", 2, 17 * 1024), ("f32", 37, 300 * 1024 + 3), ("bf16", 64, 75 * 2048 - 5),
                                               ("bf16", 9, 16 * 2048 + 9), ("bf16", 9, 20 * 2048 + 700), ("bf16", 130, 24 * 2048 + 1031),
                                               ("bf16", 3, 55 * 2048 - 1001)])
def test_rows_without_drafts_in_one_launch_and_in_two(binding, oracle, dtype, batch, vocab, greedy, beta):
    w = recipe("c4", dtype, batch=batch, k_max=0, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=64)
    inp["draft_len"] = torch.zeros(batch, dtype=torch.int32, device="cuda")
    if batch > 2:
        inp["draft_len"][batch - 2] = 1
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam,
                               beta=beta, temperature=w.temperature, draft_len=inp["draft_len"], greedy=greedy,
                               want_recovery_logprobs=batch < 64)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy,
                            want_recovery_logprobs=batch < 64)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])
    assert batch <= 2 or out["accepted_len"][batch - 2].item() == -1


# Greedy picks carry a lane's best logit as its place in a vector: the largest logit (twice, the first of them counts) at the first and
# the last place of a vector, a lane's run, a wave and the row; the largest of a row whose logits are all negative zeros and zeros.
@pytest.mark.parametrize("beta", [0.0, 0.8])
@pytest.mark.parametrize("dtype,vocab", [("bf16", 9), ("bf16", 16 * 2048 + 1), ("bf16", 40 * 2048 + 7), ("f32", 70 * 1024 + 2)])
def test_greedy_picks_the_first_of_the_largest(binding, dtype, vocab, beta):
    vec = 8 if dtype == "bf16" else 4
    edges = sorted({e % vocab for e in (0, 1, vec - 1, vec, 63 * vec, 64 * vec - 1, 256 * vec - 1, 256 * vec, 4096 * vec, vocab - 1)})
    gen = torch.Generator("cuda").manual_seed(vocab)
    rows = [torch.randn(len(edges) + 1, vocab, generator=gen, device="cuda").to(W.torch_dtype(dtype)) for _ in range(3)]
    for i, e in enumerate(edges):
        for r, v in zip(rows, (40.0, 1.0, 1.0)):
            r[i, e], r[i, vocab - 1] = v, v
    for r in rows:
        r[-1] = -0.0
        r[-1, vocab // 2:] = 0.0
    out = binding.steer_rows(*rows, torch.zeros(len(edges) + 1, device="cuda"), beta=beta, greedy=True)
    assert out["token"].tolist() == [*edges, 0]


# Rows that one token carries: its term and the row's mass hold the same rounded exponential (1.2e-7), which has to drop out of the
# log-prob.  40 others lie 22 +- 0.1 nats below it at the temperature (bf16 rounds them by up to 2^-4 of a logit): 1.1e-8 to 1.3e-8 of the
# mass, less than half a unit of the fp32 sums, and may be lost.  Without a steering term the scale is log2(e)/T rounded to fp32, repaid to
# first order: up to one unit of the exponent, 1.9e-9, more.  The store adds less than 1e-15.
@pytest.mark.parametrize("beta", [0.0, 0.8])
@pytest.mark.parametrize("dtype,batch,vocab", [("bf16", 64, 40000), ("bf16", 300, 9000), ("f32", 64, 40001), ("f32", 5, 200000)])
def test_logprob_of_a_token_that_carries_its_row(binding, dtype, batch, vocab, beta):
    gen = torch.Generator("cuda").manual_seed(batch + vocab)
    top = (torch.rand(batch, generator=gen, device="cuda") * 20 - 10).to(W.torch_dtype(dtype))
    at = torch.randint(0, vocab, (batch,), generator=gen, device="cuda")
    G = torch.full((batch, vocab), float("-inf"), device="cuda", dtype=top.dtype)
    G[:, ::vocab // 40] = (top.float() - 22 * 0.7).to(top.dtype)[:, None]
    G[torch.arange(batch), at] = top
    S = torch.zeros_like(G)
    out = binding.steer_rows(G, S, S, torch.full((batch,), 0.5, device="cuda"), beta=beta, temperature=0.7)
    lp = torch.log_softmax(G.double() / 0.7, -1)[torch.arange(batch), at]
    assert torch.equal(out["token"].long(), at)
    assert lp.max() <= -9e-9 and (out["token_logprob"].double() - lp).abs().max() <= 1.5e-8


# The draw reads its chunk by four waves, a vector a lane: a token at the first and last logit of a lane, a wave's quarter and
# a chunk and among the logits past the last vector, each with a uniform in the middle of its interval; uniforms of 0, of 1 and not
# a number, where the last token with positive probability (`keep` - 1) lies in an earlier quarter than the chunk's last.
@pytest.mark.parametrize("beta", [0.0, 0.8])
@pytest.mark.parametrize("dtype,vocab,keep", [("bf16", 2048, 2048), ("bf16", 2 * 2048 + 5, 2 * 2048 + 5), ("bf16", 4096, 4096 - 700),
                                              ("f32", 1024, 300), ("f32", 3 * 1024 + 3, 3 * 1024 + 2)])
def test_draw_at_the_edges_of_lanes_waves_and_chunks(binding, dtype, vocab, keep, beta):
    vec = 8 if dtype == "bf16" else 4
    gen = torch.Generator("cuda").manual_seed(vocab + keep)
    row = torch.randn(3, vocab, generator=gen, device="cuda").mul_(0.25).to(W.torch_dtype(dtype))
    row[0, keep:] = float("-inf")
    h = row[0].double() + beta * (row[1].double() - row[2].double())
    lp = torch.log_softmax(h, -1)
    cdf = torch.cumsum(lp.exp(), -1)
    edges = [e + d for e in (0, vec, 63 * vec, 64 * vec, 128 * vec, 192 * vec, 256 * vec, 512 * vec, keep) for d in (-1, 0)]
    want = torch.tensor([e for e in edges if 0 <= e < keep] + [0, keep - 1, keep - 1], device="cuda")
    u = (cdf[want] - 0.5 * lp[want].exp()).float()
    u[-3:] = torch.tensor([0.0, 1.0, float("nan")])
    rows = [r.expand(len(want), vocab).contiguous() for r in row]
    out = binding.steer_rows(rows[0], rows[1], rows[2], u, beta=beta)
    assert torch.equal(out["token"].long(), want)
    assert (out["token_logprob"].double() - lp[want]).abs().max() <= 1e-5


# The row pass leaves the draft token's logit as it meets it: a token at the first and last logit of a vector, a group of loads (256
# vectors), a slice and the row, and past the last vector; rows at even and odd elements, with fewer logits than a vector; one
# position more than a workgroup has groups of lanes for; a flagged sequence between two others.
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("dtype,vocab", [("bf16", 5), ("bf16", 8), ("bf16", 2048 + 3), ("bf16", 9 * 2048 + 1), ("bf16", 150 * 2048 + 7),
                                         ("f32", 3), ("f32", 1024 + 2), ("f32", 70 * 1024)])
def test_draft_logits_at_the_edges_of_vectors_groups_and_slices(binding, dtype, vocab, pad):
    vec = 8 if dtype == "bf16" else 4
    edges = sorted({e % vocab for u in (1, vec, 64 * vec, 256 * vec, 512 * vec, 1024 * vec, vocab // vec * vec) for e in (u - 1, u)}
                   | {0, vocab - 1})
    k_max = 33
    gen = torch.Generator("cuda").manual_seed(vocab)
    G, S, M = (torch.randn(3, k_max + 1, vocab + pad, generator=gen, device="cuda").mul_(3).to(W.torch_dtype(dtype))[..., :vocab]
               for _ in range(3))
    draft = torch.tensor([edges[i % len(edges)] for i in range(k_max)], dtype=torch.int32, device="cuda").repeat(3, 1)
    draft[1, 20] = vocab
    u = torch.zeros(3, k_max + 1, device="cuda")  # accepts everything
    lens = torch.tensor([k_max, k_max, 7], dtype=torch.int32, device="cuda")
    out = binding.verify_block(G, S, M, draft, u, draft_len=lens, lam=0.5, beta=0.8, want_draft_logprobs=True)
    assert out["accepted_len"].tolist() == [k_max, -1, 7]
    for b, n in ((0, k_max), (2, 7)):
        for x, T in enumerate((G, M)):
            lp = torch.log_softmax(T[b, :n].double(), -1).gather(1, draft[b, :n, None].long())[:, 0]
            assert (out["draft_logprobs"][b, :n, x].double() - lp).abs().max() <= 1e-5


# A block that fits the static scratch only without the space of the draft tokens' logits: they are gathered from the rows.
def test_draft_logits_are_gathered_where_there_is_no_space_for_them(binding, oracle):
    w = recipe("c4", "bf16", batch=400, k_max=1000, vocab=40)
    inp = W.generate(w, "cuda", seq_chunk=50)
    p = binding.make_params(400, 1000, 40, torch.bfloat16, lam=w.lam, beta=w.beta, temperature=w.temperature)
    need = binding.workspace_bytes(p)
    assert need <= binding.STATIC_SCRATCH_BYTES < need + 400 * 1000 * 8
    inp["draft_len"] = torch.tensor([(37 * i) % 1001 for i in range(400)], dtype=torch.int32, device="cuda")
    inp["draft"][2, 0] = 40  # flagged
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, draft_len=inp["draft_len"], want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, want_recovery_logprobs=False,
                            num_threads=8)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])
    assert out["accepted_len"][2].item() == -1


# Draft slots and rows behind a sequence's length are the caller's: ids there are outside the vocabulary, rows not a number.  Ids outside
# the vocabulary at the first and the last valid slot flag their sequence.  With a pair of lanes' groups to every position and
# with rounds, in one window and two, with the space of the draft tokens' logits and (24000 sequences) without it.
@pytest.mark.parametrize("batch,k_max,vocab", [(3, 1, 5), (5, 8, 3001), (5, 9, 3001), (3, 32, 40001), (6, 33, 3001), (300, 16, 801),
                                               (300, 17, 801), (64, 20, 104900), (24000, 16, 40), (24000, 16, 700)])
def test_slots_behind_the_length_are_ignored_and_ids_outside_the_vocabulary_flag(binding, oracle, batch, k_max, vocab):
    w = recipe("c4", "bf16", batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=16 if vocab > 4000 else 600)
    gen = torch.Generator("cuda").manual_seed(batch + k_max)
    lens = torch.randint(0, k_max + 1, (batch,), generator=gen, device="cuda", dtype=torch.int32)
    lens[0], lens[1], lens[2] = k_max, k_max, 1
    behind = torch.arange(k_max, device="cuda") >= lens[:, None]
    odd = torch.tensor([-1, vocab, -2**31, 2**31 - 1, vocab + 1], dtype=torch.int32, device="cuda")
    inp["draft"] = torch.where(behind, odd.repeat(batch * k_max // 5 + 1)[:batch * k_max].view(batch, k_max), inp["draft"])
    for k in ("G", "S_ctx", "S_noctx"):
        for t in range(1, k_max + 1):
            inp[k][lens < t, t] = float("nan")
    inp["draft"][1, k_max - 1], inp["draft"][2, 0] = vocab, -1
    inp["draft_len"] = lens
    if batch == 24000:
        p = binding.make_params(batch, k_max, vocab, torch.bfloat16, lam=w.lam, beta=w.beta, temperature=w.temperature)
        assert binding.workspace_bytes(p) <= binding.STATIC_SCRATCH_BYTES < binding.workspace_bytes(p) + batch * k_max * 8
        assert binding.first_window(p) == (4 if vocab == 700 else 16)
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, draft_len=lens)
    assert out["accepted_len"][1:3].tolist() == [-1, -1]
    assert (out["accepted_len"] >= 0).sum().item() == batch - 2
    seqs = torch.arange(0, batch, max(1, batch // 300), device="cuda")
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, seqs=seqs, want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], lens, seqs=seqs)
    if batch < 24000:
        staged = in_stages(binding, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, draft_len=lens)
        parity.compare(staged, ora, inp["uniforms"], lens, seqs=seqs)


# A ragged batch's rows are looked up 64 sequences at a time from the last row's on: runs of 61 .. 129 sequences without a row
# between two that have some, at the start and at the end; rows of one slice and of several, fewer of them than waves and more.
@pytest.mark.parametrize("vocab", [40, 33 * 2048 + 3])
@pytest.mark.parametrize("full", [(0, 63, 64, 126, 255), (64, 129, 258, 300), (130, 131), (0,), (299,)])
def test_row_lookup_over_sequences_without_rows(binding, oracle, vocab, full):
    w = recipe("c4", "bf16", batch=301, k_max=4, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=64)
    lens = torch.zeros(301, dtype=torch.int32, device="cuda")
    for i, b in enumerate(full):
        lens[b] = 1 + i % 4
    inp["draft_len"] = lens
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, draft_len=lens, want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], lens)


# The same over thousands of sequences without rows, in LDS (up to 8192 sequences) and in global memory: runs of 63 .. 65 x 64 sequences
# and one more or less, rows that only the first or the last sequence has.
@pytest.mark.parametrize("batch", [8192, 8193, 20011])
@pytest.mark.parametrize("full", [(0, 64, 65, 4096, 4160, 4161, 8191), (0,), (-1,), (63, 4095, 4097, -2), (1, 128, 129, -65, -64, -1)])
def test_row_lookup_over_thousands_of_sequences_without_rows(binding, oracle, batch, full):
    w = recipe("c4", "bf16", batch=batch, k_max=2, vocab=9)
    inp = W.generate(w, "cuda", seq_chunk=4096)
    at = torch.tensor([b % batch for b in full], device="cuda")
    lens = torch.zeros(batch, dtype=torch.int32, device="cuda")
    lens[at] = torch.arange(len(full), dtype=torch.int32, device="cuda") % 2 + 1
    inp["draft_len"] = lens
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, draft_len=lens, want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, seqs=at, want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], lens, seqs=at)
    assert torch.all((out["draft_logprobs"] == 0).all(-1) == (torch.arange(2, device="cuda") >= lens[:, None]))


# Shared rows whose parts have 1 .. 9 chunks over after whole rounds of 16, dealt out in quarters (1 .. 4), halves (5 .. 8) or whole: of
# the last part, which may have fewer, the logits past the last vector and a last chunk of one vector among them.
@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0)])
@pytest.mark.parametrize("dtype,batch,chunks,more", [("bf16", 64, 75, -5), ("bf16", 64, 67, 8), ("bf16", 100, 42, 0), ("bf16", 127, 43, 1),
                                                     ("bf16", 128, 36, 9), ("f32", 128, 49, 2), ("f32", 90, 35, 4)])
def test_chunks_over_are_dealt_out(binding, oracle, dtype, batch, chunks, more, greedy, beta):
    vocab = chunks * (2048 if dtype == "bf16" else 1024) + more
    w = recipe("c4", dtype, batch=batch, k_max=2, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=32)
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=beta,
                               temperature=w.temperature, draft_len=inp["draft_len"], greedy=greedy)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy,
                            want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])


# Row-pass slices merged by 16 lanes: 1, 15 .. 17 and 64 slices (the most) of a row, with a remainder.
@pytest.mark.parametrize("dtype,vocab", [("bf16", 2048), ("bf16", 15 * 2048 + 1), ("bf16", 16 * 2048), ("bf16", 17 * 2048 + 7),
                                         ("bf16", 64 * 2048), ("f32", 63 * 1024 + 1)])
def test_slice_merge_edges(binding, oracle, dtype, vocab):
    w = recipe("c2", dtype, batch=2, k_max=9, vocab=vocab)
    inp = W.generate(w, "cuda")
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam,
                               beta=w.beta, temperature=w.temperature, want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], None)
    parity.compare(in_stages(binding, inp, lam=w.lam, beta=w.beta, temperature=w.temperature), ora, inp["uniforms"], None)


# Windows of 1, 1, 2, ... positions, at the fewest bytes a position that get them (240 MiB, 280 with 4 and 5
# positions): 4, 5, 6 and 8 positions end in windows of 2, 3 (no short last window), 2 and 4.  Every length occurs, and one
# flagged sequence of each kind.
@pytest.mark.parametrize("k_max,greedy", [(4, False), (5, True), (6, False), (8, False)])
def test_doubling_windows_equal_the_one_pass_schedule(binding, oracle, k_max, greedy):
    w = recipe("c2" if k_max == 6 else "c5", "bf16", batch=1000, k_max=k_max, vocab=73401 if k_max < 6 else 63001)
    inp = W.generate(w, "cuda", seq_chunk=40)
    p = binding.make_params(w.batch, k_max, w.vocab, torch.bfloat16, lam=w.lam, beta=w.beta, temperature=w.temperature)
    assert binding.first_window(p) == 1
    lens = torch.randint(0, k_max + 1, (w.batch,), generator=torch.Generator("cuda").manual_seed(k_max), device="cuda",
                         dtype=torch.int32)
    lens[7], lens[8] = k_max + 1, -1
    lens[9] = k_max
    inp["draft"][9, k_max - 1] = w.vocab  # out of the vocabulary, behind the first window
    inp["draft_len"] = lens
    kw = dict(lam=w.lam, beta=w.beta, temperature=w.temperature, draft_len=lens, greedy=greedy)
    args = [inp[k] for k in ("G", "S_ctx", "S_noctx", "draft", "uniforms")]
    got = binding.verify_block(*args, **kw)
    one = binding.verify_block(*args, full_rows=True, **kw)
    for k in ("accepted_len", "next_token", "next_token_logprob"):
        assert torch.equal(torch.nan_to_num(got[k]), torch.nan_to_num(one[k])), k
    assert got["accepted_len"][7:10].tolist() == [-1, -1, -1]
    n = got["accepted_len"]
    seqs = torch.arange(0, w.batch, 20, device="cuda")
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, seqs=seqs, greedy=greedy,
                            want_recovery_logprobs=False)
    parity.compare(got, ora, inp["uniforms"], lens, seqs=seqs)
    for lo in (1, 2):  # rows behind the window a sequence was rejected in are never read
        out = (n >= 0) & (n < lo) & (lens > lo)
        assert out.any()
        for k in ("G", "S_noctx"):
            inp[k][out, lo:] = float("nan")
    again = binding.verify_block(*args, **kw)
    for k in ("accepted_len", "next_token", "next_token_logprob"):
        assert torch.equal(torch.nan_to_num(got[k]), torch.nan_to_num(again[k])), k


# bf16 rows off 4-byte boundaries are read from one element before their start, which is masked: an odd stride puts
# every other row there.  The padding (and so the element before a row) is NaN.  Sizes around a vector, a chunk and
# a slice; `shift` moves G alone (its rows then differ in parity from the specialists').
@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0)])
@pytest.mark.parametrize("vocab,pad,shift", [(6, 1, 0), (7, 2, 0), (8, 1, 0), (9, 0, 0), (2047, 0, 0), (2048, 1, 0), (2049, 2, 0),
                                             (16384, 3, 0), (16391, 0, 0), (16391, 0, 1), (16384, 3, 1), (9, 2, 1)])
def test_rows_at_odd_elements(binding, oracle, vocab, pad, shift, greedy, beta):
    w = recipe("c4", "bf16", batch=6, k_max=3, vocab=vocab + pad)
    inp = W.generate(w, "cuda")
    for k in ("G", "S_ctx", "S_noctx"):
        inp[k][..., vocab:] = float("nan")
        if k == "G" and shift:
            flat = torch.full((inp[k].numel() + 1,), float("nan"), dtype=torch.bfloat16, device="cuda")
            flat[1:].copy_(inp[k].reshape(-1))
            inp[k] = flat[1:].view_as(inp[k])
        inp[k] = inp[k][..., :vocab]
    inp["draft"] = inp["draft"].clamp(max=vocab - 1)
    inp["draft_len"] = torch.tensor([3, 0, 1, 2, 3, 2], dtype=torch.int32, device="cuda")
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=beta,
                               temperature=w.temperature, draft_len=inp["draft_len"], greedy=greedy,
                               want_recovery_logprobs=True, want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])


def test_row_modes_take_every_form_of_rows_the_block_takes(binding):
    """steer_rows and sample_rows hand pointers over themselves: padded rows, a single row cut from a wider tensor,
    specialist logits of another shape, uniforms of another type, shape or device must give what the block gives."""
    w = recipe("c4", "bf16", batch=4, k_max=1, vocab=3001)
    inp = W.generate(w, "cuda")
    wide = {k: torch.cat([inp[k].view(8, 3001), torch.full((8, 7), float("nan"), dtype=torch.bfloat16, device="cuda")], 1)
            for k in ("G", "S_ctx", "S_noctx")}
    u = inp["uniforms"].reshape(8)
    flat = [inp[k].view(8, 3001) for k in ("G", "S_ctx", "S_noctx")]
    want = binding.verify_block(*(t.view(8, 1, 3001) for t in flat), torch.empty(8, 0, dtype=torch.int32, device="cuda"),
                                u.view(8, 1), beta=0.7, temperature=0.9, want_recovery_logprobs=True)
    kw = dict(beta=0.7, temperature=0.9, want_logprobs=True)
    padded = [wide[k][:, :3001] for k in ("G", "S_ctx", "S_noctx")]
    for rows, un in ((flat, u), (padded, u.double()), ([flat[0], inp["S_ctx"], inp["S_noctx"]], u.view(2, 4)), (flat, u.cpu())):
        got = binding.steer_rows(*rows, un, **kw)
        # padded rows start at other offsets: the sums of a row at an odd element are grouped differently
        assert torch.equal(got["token"], want["next_token"])
        assert torch.allclose(got["token_logprob"], want["next_token_logprob"], rtol=0, atol=2e-6)
        assert torch.allclose(got["logprobs"], want["recovery_logprobs"], rtol=0, atol=4e-6)
    one = binding.steer_rows(padded[0][3:4], flat[1][3:4], padded[2][3:4], u[3:4], **kw)
    assert one["token"].item() == want["next_token"][3].item()
    for bad in ((flat[0], flat[1], flat[2][:, ::2]), (flat[0], flat[1].float(), flat[2]), (flat[0], padded[1], flat[2])):
        with pytest.raises((ValueError, RuntimeError)):
            binding.steer_rows(*bad, u, **kw)
    with pytest.raises(ValueError):
        binding.steer_rows(*(t.cpu() for t in flat), u, **kw)


def test_doubling_windows_inside_a_hip_graph(binding):
    """The launches of several windows captured once and replayed on new drafts, lengths and uniforms, with eager
    calls on the same workspace between the replays; every replay equals the direct call."""
    w = recipe("c5", "bf16", batch=1000, k_max=5, vocab=73401)
    inp = W.generate(w, "cuda", seq_chunk=40)
    inp["draft_len"] = torch.randint(0, 6, (1000,), device="cuda", dtype=torch.int32)
    p = binding.make_params(1000, 5, w.vocab, torch.bfloat16, lam=w.lam, beta=w.beta, temperature=w.temperature)
    assert binding.first_window(p) == 1
    ws = torch.empty(binding.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    outs = [[torch.empty(1000, dtype=dt, device="cuda") for dt in (torch.int32, torch.int32, torch.float32)] for _ in range(2)]

    def call(out):
        binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["draft_len"], inp["uniforms"], p,
                                 *out, None, None, ws)

    call(outs[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(outs[0])
    for rnd in range(4):
        gen = torch.Generator("cuda").manual_seed(rnd)
        inp["uniforms"].uniform_(generator=gen)
        inp["draft_len"].random_(0, 6, generator=gen)
        inp["draft"].copy_(inp["draft"].roll(1, 0))
        for t in outs[0]:
            t.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        call(outs[1])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(*outs)), rnd
        assert torch.all(outs[0][0] >= 0)


def test_edge_resample_on_columns_of_a_wider_payload(binding):
    """The first 16 columns of a top-32 payload, handed over as a view, give what a copy of them gives."""
    w = recipe("c4", "bf16", batch=9, k_max=2, vocab=4099)
    inp = W.generate(w, "cuda")
    row = torch.randint(0, 3, (9,), generator=torch.Generator("cuda").manual_seed(3), device="cuda", dtype=torch.int32)
    idx, val = binding.cloud_topk(inp["G"], inp["S_noctx"], row, beta=w.beta, topk=32)
    u = inp["uniforms"][:, -1].contiguous()
    copies = idx[:, :16].contiguous(), val[:, :16].contiguous()
    want = binding.edge_resample(*copies, inp["S_ctx"], row, u, beta=w.beta, temperature=w.temperature)
    got = binding.edge_resample(idx[:, :16], val[:, :16], inp["S_ctx"], row, u, beta=w.beta, temperature=w.temperature)
    for k in ("next_token", "next_token_logprob"):
        assert torch.equal(got[k], want[k]), k


# Rows that are all odd although every stride is even (each tensor starts one element late), and the same rows at even
# elements, on both sides of a whole number of chunks: the launch is planned with the chunks its rows have.
@pytest.mark.parametrize("vocab", [4 * 2048 - 2, 4 * 2048, 4 * 2048 + 2])
@pytest.mark.parametrize("late", [0, 1])
def test_odd_bases_with_even_strides(binding, oracle, vocab, late):
    w = recipe("c4", "bf16", batch=3, k_max=2, vocab=vocab)
    inp = W.generate(w, "cuda")
    for k in ("G", "S_ctx", "S_noctx"):
        flat = torch.full((inp[k].numel() + 2,), float("nan"), dtype=torch.bfloat16, device="cuda")
        flat[late:late + inp[k].numel()].copy_(inp[k].reshape(-1))
        inp[k] = flat[late:late + inp[k].numel()].view_as(inp[k])
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, draft_len=inp["draft_len"], want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"])
    staged = in_stages(binding, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, draft_len=inp["draft_len"])
    parity.compare(staged, ora, inp["uniforms"], inp["draft_len"])


# Ratio test: 16 lanes to a (position, tensor) pair.  As many pairs as a workgroup has such groups (8 positions with 4 waves, 32
# with 16) and one position more, which takes rounds; verdicts of 5 .. 8 (two waves) and of more positions (eight).
@pytest.mark.parametrize("batch,k_max,vocab", [(2, 8, 3001), (2, 9, 3001), (2, 32, 3001), (2, 33, 3001), (2, 32, 40001), (2, 33, 40001),
                                               (300, 16, 801), (300, 17, 801), (64, 20, 104900), (64, 36, 58301)])
def test_ratio_test_rounds(binding, oracle, batch, k_max, vocab):
    w = recipe("c3", "bf16", batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=16)
    gen = torch.Generator("cuda").manual_seed(k_max)
    lens = torch.randint(0, k_max + 1, (batch,), generator=gen, device="cuda", dtype=torch.int32)
    lens[0] = k_max
    lens[-1] = k_max
    inp["draft"][-1, k_max - 1] = vocab  # flagged by the last position
    inp["draft_len"] = lens
    args = [inp[k] for k in ("G", "S_ctx", "S_noctx", "draft", "uniforms")]
    kw = dict(lam=w.lam, beta=w.beta, temperature=w.temperature, draft_len=lens)
    got = binding.verify_block(*args, **kw)
    one = binding.verify_block(*args, full_rows=True, want_draft_logprobs=True, **kw)
    for k in ("accepted_len", "next_token", "next_token_logprob"):
        assert torch.equal(torch.nan_to_num(got[k]), torch.nan_to_num(one[k])), k
    assert got["accepted_len"][-1].item() == -1
    seqs = torch.arange(0, batch, max(1, batch // 8), device="cuda")
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, seqs=seqs, want_recovery_logprobs=False)
    parity.compare(one, ora, inp["uniforms"], lens, seqs=seqs)
    parity.compare(in_stages(binding, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, draft_len=lens), ora, inp["uniforms"], lens, seqs=seqs)


# The same launch by chunks and drafts: up to 16 chunks it is one workgroup or several by the number of drafts, beyond them
# two 16-wave parts (33 drafts).  Without a draft there are no counters: one workgroup takes its row whole.
@pytest.mark.parametrize("dtype,k_max,chunks", [("bf16", 0, 4), ("bf16", 0, 9), ("bf16", 0, 16), ("f32", 0, 17), ("bf16", 9, 4), ("f32", 8, 8),
                                                ("bf16", 16, 9), ("bf16", 17, 16), ("bf16", 32, 17), ("f32", 33, 17)])
@pytest.mark.parametrize("greedy", [False, True])
def test_recovery_launch_by_chunks_and_drafts(binding, oracle, dtype, k_max, chunks, greedy):
    w = recipe("c3", dtype, batch=3, k_max=k_max, vocab=chunks * (2048 if dtype == "bf16" else 1024))
    inp = W.generate(w, "cuda")
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, greedy=greedy, want_draft_logprobs=True)
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, greedy=greedy,
                            want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], None)
    parity.compare(in_stages(binding, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, greedy=greedy), ora, inp["uniforms"], None)


# Row pass in slices of one group of loads (256 vectors), of which a row's last holds 1 to 255 vectors, and of two (500 sequences, the first two sizes): at the edges
# of its two or four loads, with logits past the last vector and without, rows at odd elements, and the draft tokens' logits in that slice.
@pytest.mark.parametrize("batch", [200, 500])
@pytest.mark.parametrize("dtype,vocab", [(dt, (8 if dt == "bf16" else 4) * (256 * groups + more) + rest) for dt, groups, more, rest in (
    ("bf16", 15, 160, 0), ("bf16", 14, 66, 1), ("bf16", 3, 1, 0), ("bf16", 3, 63, 3), ("bf16", 3, 64, 0), ("bf16", 3, 65, 0), ("bf16", 0, 127, 5), ("bf16", 2, 128, 0), ("bf16", 0, 130, 1), ("bf16", 1, 192, 0), ("bf16", 2, 255, 7),
    ("f32", 3, 1, 0), ("f32", 2, 64, 3), ("f32", 0, 65, 2), ("f32", 1, 128, 1), ("f32", 0, 129, 0), ("f32", 1, 255, 1))])
def test_row_pass_at_the_end_of_short_slices(binding, oracle, dtype, vocab, batch):
    k_max = 4
    w = recipe("c4", dtype, batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda")
    last = torch.arange(batch, device="cuda", dtype=torch.int32)
    inp["draft"][:, 1] = vocab - 1 - last % min(vocab, 1200)
    out = binding.verify_block(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["uniforms"], lam=w.lam, beta=w.beta,
                               temperature=w.temperature, want_draft_logprobs=True)
    inp["draft_len"] = torch.full((batch,), k_max, dtype=torch.int32, device="cuda")
    seqs = torch.arange(0, batch, 7, device="cuda")
    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=w.beta, temperature=w.temperature, seqs=seqs, want_recovery_logprobs=False)
    parity.compare(out, ora, inp["uniforms"], inp["draft_len"], seqs=seqs)


# Small blocks in one launch: a wave a chunk of 256 vectors, four to a workgroup.  Rows shorter than a vector, of one chunk and one logit more
# and less, of whole workgroups and a chunk over, the longest (64 chunks, the last one whole, partial or of logits past the last vector)
# and, beyond and where the space does not suffice (16 greedy drafts), two launches; rows at odd elements; lengths of 0, ids and
# lengths that flag.  On a space of garbage that the calls before have left, direct and as the stages of the timed call, whose tokens are the
# same.  Behind each size the modes that take one launch: sampled, greedy, and both without steering; a CPU test holds them against the rule.
ONCE_SIZES = [
    ("bf16", 3, 2, 5, "sS"), ("bf16", 5, 16, 7, "sS"), ("bf16", 5, 3, 2047, "sS"), ("bf16", 5, 4, 2048, "sS"), ("bf16", 5, 1, 2049, "sS"),
    ("bf16", 3, 4, 4 * 2048 + 9, "sS"), ("bf16", 3, 4, 5 * 2048 + 9, "sgSG"), ("bf16", 5, 3, 7 * 2048 + 1, "sgSG"), ("bf16", 3, 16, 17 * 2048 - 3, "sS"), ("bf16", 6, 4, 32000, "sgSG"), ("bf16", 1, 8, 64 * 2048, "sgSG"),
    ("bf16", 4, 2, 64 * 2048 - 1, ""), ("bf16", 4, 2, 64 * 2048 - 8, "sgSG"), ("bf16", 4, 2, 63 * 2048 + 5, "sgSG"), ("bf16", 2, 3, 64 * 2048 + 1, ""),
    ("bf16", 40, 2, 3 * 2048 + 1, "sS"), ("f32", 1, 4, 32000, "sgSG"), ("f32", 4, 4, 1025, "sSG"), ("f32", 4, 4, 5 * 1024 + 1, "sgSG"), ("f32", 3, 16, 33 * 1024 + 2, "sS"),
    ("f32", 2, 2, 64 * 1024, "sgSG"), ("f32", 25, 3, 40000, "sS"), ("bf16", 24, 3, 32 * 2048, "sS")]


@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0), (True, 0.0)])
@pytest.mark.parametrize("dtype,batch,k_max,vocab", [c[:4] for c in ONCE_SIZES])
def test_small_blocks_in_one_launch(binding, oracle, dtype, batch, k_max, vocab, greedy, beta):
    w = recipe("c4", dtype, batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda")
    gen = torch.Generator("cuda").manual_seed(batch + vocab)
    lens = torch.randint(0, k_max + 1, (batch,), generator=gen, device="cuda", dtype=torch.int32)
    lens[0] = k_max
    if batch > 3:
        lens[1], lens[2], lens[3] = k_max + 1, 0, 1
        inp["draft"][3, 0] = vocab
    inp["draft_len"] = lens
    p = binding.make_params(batch, k_max, vocab, W.torch_dtype(dtype), lam=w.lam, beta=beta, temperature=w.temperature,
                            flags=binding.SS_FLAG_GREEDY if greedy else 0)
    ws = torch.full((binding.workspace_bytes(p),), 0xAB, dtype=torch.uint8, device="cuda")
    names = ("accepted_len", "next_token", "next_token_logprob", "recovery_logprobs", "draft_logprobs")

    def call(timed):
        mk = lambda dt, *shape: torch.full(shape, -7, dtype=dt, device="cuda")
        o = [mk(torch.int32, batch), mk(torch.int32, batch), mk(torch.float32, batch), None, mk(torch.float32, batch, k_max, 2)]
        binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], lens, inp["uniforms"], p, *o, ws, timed=timed)
        torch.cuda.synchronize()
        return dict(zip(names, o))

    ora = parity.oracle_run(oracle, inp, lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy, want_recovery_logprobs=False)
    first = call(False)
    parity.compare(first, ora, inp["uniforms"], lens)
    staged, again = call(True), call(False)
    for k in ("accepted_len", "next_token", "next_token_logprob"):
        assert torch.equal(torch.nan_to_num(first[k]), torch.nan_to_num(staged[k])), k
    # their sums are grouped by chunks here and by slices there: each is within the bound to the oracle, so twice that apart
    assert torch.allclose(first["draft_logprobs"], staged["draft_logprobs"], rtol=0, atol=2 * parity.LOGPROB_ATOL, equal_nan=True)
    assert all(first[k] is None or torch.equal(torch.nan_to_num(first[k]), torch.nan_to_num(again[k])) for k in names)


# The same launch on rows at odd elements of some of the three tensors (`late`: those that begin one element late; without steering S_noctx
# is read at G's parity whatever its own), with tokens masked by the generalist, whole chunks of them, by all three models and by the
# specialist alone, a drafted one among them, and NaN in every row that has no say: those behind a length, and S_ctx but for the recovery row.
ONCE_FORM_SIZES = [("bf16", 4, 3, 9 * 2048 + 7, "sgSG"), ("bf16", 4, 3, 9 * 2048 + 8, "sgSG"), ("f32", 4, 3, 9 * 1024 + 3, "sgSG")]


@pytest.mark.parametrize("greedy,beta", [(False, 0.8), (True, 0.8), (False, 0.0), (True, 0.0)])
@pytest.mark.parametrize("late", ["", "G", "S_noctx", "G S_ctx", "G S_noctx", "G S_ctx S_noctx"])
@pytest.mark.parametrize("dtype,batch,k_max,vocab", [c[:4] for c in ONCE_FORM_SIZES])
def test_small_blocks_in_one_launch_of_odd_and_masked_rows(binding, oracle, dtype, batch, k_max, vocab, late, greedy, beta):
    w = recipe("c4", dtype, batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda")
    lens = torch.tensor([3, 0, 2, 3], dtype=torch.int32, device="cuda")
    inp["draft_len"] = lens
    gen = torch.Generator("cuda").manual_seed(vocab)
    chunk = vocab // 9
    common, alone, spec = (torch.rand(inp["G"].shape, generator=gen, device="cuda") < x for x in (0.2, 0.2, 0.1))
    common[:, :, chunk:2 * chunk] = True
    alone[:, 1:, 5 * chunk:6 * chunk] = True
    at = torch.arange(batch, device="cuda").view(-1, 1), torch.arange(k_max, device="cuda").view(1, -1), inp["draft"].long()
    for m in (common, alone, spec):
        m[at] = False
    alone[0, 1, inp["draft"][0, 1]] = True
    inp["uniforms"][0, :2] = torch.tensor([0.0, 0.5], device="cuda")  # rejected there
    inp["uniforms"][3, :3] = 0.0                                      # all accepted
    inp["G"][common | alone] = float("-inf")
    for k in ("S_ctx", "S_noctx"):
        inp[k][common | spec] = float("-inf")
    kw = dict(lam=w.lam, beta=beta, temperature=w.temperature, greedy=greedy)
    ora = parity.oracle_run(oracle, inp, want_recovery_logprobs=False, **kw)
    for k in ("G", "S_ctx", "S_noctx"):
        for b, n in enumerate(lens.tolist()):
            inp[k][b, n + 1:] = float("nan")
            if k == "S_ctx":
                inp[k][b, torch.arange(k_max + 1, device="cuda") != int(ora["accepted_len"][b])] = float("nan")
        flat = torch.full((inp[k].numel() + 8,), float("nan"), dtype=inp[k].dtype, device="cuda")
        o = int(k in late.split())
        flat[o:o + inp[k].numel()] = inp[k].flatten()
        inp[k] = flat[o:o + inp[k].numel()].view_as(inp[k])
    one = binding.verify_block(*(inp[k] for k in ("G", "S_ctx", "S_noctx", "draft", "uniforms")), draft_len=lens, want_draft_logprobs=True, **kw)
    assert one["accepted_len"].tolist()[::3] == [1, 3]
    parity.compare(one, ora, inp["uniforms"], lens)
    parity.compare(in_stages(binding, inp, draft_len=lens, **kw), ora, inp["uniforms"], lens)


# Without steering the bonus position asks for nothing but the generalist's row: S_noctx ends behind its k_max rows here (what follows
# belongs to someone else), with logits past the last vector of a row and without, all drafts accepted.
@pytest.mark.parametrize("greedy", [False, True])
@pytest.mark.parametrize("dtype,vocab", [("bf16", 5), ("bf16", 2 * 2048 + 9), ("bf16", 4096), ("f32", 1027), ("f32", 32000)])
def test_without_steering_the_bonus_row_of_the_specialist_is_not_asked_for(binding, oracle, dtype, vocab, greedy):
    w = recipe("c4", dtype, batch=1, k_max=3, vocab=vocab)
    inp = W.generate(w, "cuda")
    inp["uniforms"][:, :3] = 0.0
    inp["draft_len"] = None
    want = parity.oracle_run(oracle, inp, lam=w.lam, beta=0.0, temperature=w.temperature, greedy=greedy, want_recovery_logprobs=False)
    inp["S_noctx"][:, 3] = float("nan")
    kw = dict(lam=w.lam, beta=0.0, temperature=w.temperature, greedy=greedy)
    got = binding.verify_block(*(inp[k] for k in ("G", "S_ctx", "S_noctx", "draft", "uniforms")), want_draft_logprobs=True, **kw)
    assert got["accepted_len"].item() == 3
    parity.compare(got, want, inp["uniforms"], None)


ONCE_GRAPH_SIZES = [("f32", 1, 4, 32000, "sg"), ("bf16", 4, 4, 50257, "sg")]


@pytest.mark.parametrize("greedy", [False, True])
@pytest.mark.parametrize("dtype,batch,k_max,vocab", [c[:4] for c in ONCE_GRAPH_SIZES])
def test_small_blocks_in_one_launch_inside_a_hip_graph(binding, dtype, batch, k_max, vocab, greedy):
    """The words of a captured call carry the same tag on every replay: replays on new drafts, lengths and uniforms, one behind the
    other and with direct calls on the same workspace between them, equal the direct calls."""
    w = recipe("c4", dtype, batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda")
    inp["draft_len"] = torch.full((batch,), k_max, dtype=torch.int32, device="cuda")
    p = binding.make_params(batch, k_max, vocab, W.torch_dtype(dtype), lam=w.lam, beta=w.beta, temperature=w.temperature,
                            flags=binding.SS_FLAG_GREEDY if greedy else 0)
    ws = torch.full((binding.workspace_bytes(p),), 0x5A, dtype=torch.uint8, device="cuda")
    outs = [[torch.empty(batch, dtype=dt, device="cuda") for dt in (torch.int32, torch.int32, torch.float32)] for _ in range(2)]

    def call(out):
        binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], inp["draft_len"], inp["uniforms"], p,
                                 *out, None, None, ws)

    call(outs[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(outs[0])
    for rnd in range(24):
        gen = torch.Generator("cuda").manual_seed(rnd)
        inp["uniforms"].uniform_(generator=gen)
        inp["draft_len"].random_(0, k_max + 1, generator=gen)
        inp["draft"].copy_(inp["draft"].roll(1, 1))
        inp["S_noctx"].copy_(inp["S_noctx"].roll(1, 2))
        for t in outs[0]:
            t.fill_(-7)
        g.replay()
        if rnd % 3:  # else the next replay follows this one's clearing with nothing between
            torch.cuda.synchronize()
            call(outs[1])
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(*outs)), rnd
        assert torch.all(outs[0][0] >= 0)


# The cloud top-k queues what reaches its bound wave by wave: as many equal largest logits as its buffers hold (256 in registers,
# 1024 candidates, 2048 vectors) and one more or less, next to each other, a vector apart and all in the lanes of one wave.
@pytest.mark.parametrize("spread", ["dense", "vectors", "one wave"])
@pytest.mark.parametrize("dtype,count", [("bf16", 31), ("bf16", 255), ("bf16", 257), ("bf16", 1024), ("bf16", 1025), ("f32", 1023),
                                         ("f32", 2048), ("f32", 2049)])
def test_topk_of_equal_logits_fills_its_buffers(binding, dtype, count, spread):
    vec, vocab, k = (8, 70007, 64) if dtype == "bf16" else (4, 50001, 64)
    at = torch.arange(count, device="cuda")
    if spread == "vectors":
        at = at * vec % (vocab - vec) + at * vec // (vocab - vec)
    elif spread == "one wave":  # 64 lanes x vec logits, 1024 vectors on for the next ones
        at = at % (64 * vec) + at // (64 * vec) * 1024 * vec
    at = at[at < vocab].unique()
    gen = torch.Generator("cuda").manual_seed(count)
    G = torch.rand(2, 1, vocab, generator=gen, device="cuda").mul_(3).to(W.torch_dtype(dtype))
    M = torch.zeros_like(G)
    G[0, 0, at] = 5.0
    h = (G.double() - 0.5 * M.double())[:, 0]
    value, index = torch.sort(h, dim=-1, descending=True, stable=True)
    got_i, got_v = binding.cloud_topk(G, M, torch.zeros(2, dtype=torch.int32, device="cuda"), beta=0.5, topk=k)
    assert torch.equal(got_i.long(), index[:, :k]) and torch.equal(got_v, value[:, :k].float())


# A workspace that lacks the space of the draft tokens' logits (more than 512 positions): they are gathered, with the same outputs bit
# for bit, and nothing is written behind it; in one window and several, with shared recovery rows and with one workgroup each.
@pytest.mark.parametrize("batch,k_max,vocab", [(1, 513, 3001), (27, 19, 40001), (128, 5, 70000), (300, 17, 801), (64, 20, 104900)])
def test_a_workspace_without_space_for_the_draft_logits(binding, batch, k_max, vocab):
    w = recipe("c4", "bf16", batch=batch, k_max=k_max, vocab=vocab)
    inp = W.generate(w, "cuda", seq_chunk=16)
    lens = torch.randint(0, k_max + 1, (batch,), generator=torch.Generator("cuda").manual_seed(batch), device="cuda", dtype=torch.int32)
    lens[0] = k_max
    if batch > 2:
        inp["draft"][0, k_max - 1] = vocab  # flagged by its last position
    p = binding.make_params(batch, k_max, vocab, torch.bfloat16, lam=w.lam, beta=w.beta, temperature=w.temperature)
    need = binding.workspace_bytes(p)
    lean = need - (8 * batch * k_max + 255) // 256 * 256
    outs = []
    for n in (need, lean):
        ws = torch.full((need + 256,), 0xAB, dtype=torch.uint8, device="cuda")
        out = [torch.full((batch,), -7, dtype=dt, device="cuda") for dt in (torch.int32, torch.int32, torch.float32)]
        binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], lens, inp["uniforms"], p, *out, None, None, ws[:n])
        assert torch.all(ws[n:] == 0xAB)
        outs.append(out)
    assert all(torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)) for a, b in zip(*outs))
    assert (outs[0][0] >= 0).sum().item() == batch - (batch > 2)
    with pytest.raises(binding.SpecSteerError):
        binding.verify_block_raw(inp["G"], inp["S_ctx"], inp["S_noctx"], inp["draft"], lens, inp["uniforms"], p, *outs[1], None, None, ws[:lean - 256])
