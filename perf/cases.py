"""The calls that stand for this framework's use, each through its public entry points.

A case is one call (or, for the deployment split, the cloud and the edge half of one) on logits that are
already in HBM.  Sizes and input recipes are those of ``paper_2603_16219_amd.workloads`` (c1 .. c5), of the
benchmark's other modes, and of the tests (an odd vocabulary, fp32 logits, greedy decoding, log-prob rows).

What is measured, and the ranges behind it (``draw``):
  batch 1 .. 512 sequences, draft length 1 .. 16, vocabulary 32000 .. 256000 (odd ones among them), bf16 and
  fp32, ragged and full drafts, sampled and greedy, per-position log-probs and recovery rows, always-on
  steering and plain sampling of 1 .. 4352 rows, top-8 .. top-64 downlink of 1 .. 512 rows.
"""
from __future__ import annotations

import math

import torch

from paper_2603_16219_amd import binding
from paper_2603_16219_amd.workloads import WORKLOADS

LAMBDA = 0.5  # the paper's default threshold
# Mean probability that one position of a recipe is accepted at that threshold (the recipes' own tests pin
# about 0.8 for c1 .. c4 and 0.4 for c5): work() needs it, since the rows behind a first rejection are not
# among the bytes that the algorithm cannot do without.
ACCEPT = {"c1": 0.8, "c2": 0.8, "c3": 0.8, "c4": 0.8, "c5": 0.4}
MAX_ROWS = 4352  # rows of the largest steering / sampling call: 256 sequences of 17 rows
MAX_STATE_BYTES = 3 * 512 * 9 * 256000 * 2  # the largest listed state


def listed():
    return [
        # One interactive user: a single short block, the smallest call; only launches and latency count.
        dict(name="c1_one_user", op="verify", recipe="c1", batch=1, k_max=4, vocab=32000, dtype="f32", ragged=False,
             greedy=False),
        # A handful of users on a 152k vocabulary: 46 MB, still mostly latency.
        dict(name="c2_few_users", op="verify", recipe="c2", batch=8, k_max=8, vocab=151936, dtype="bf16",
             ragged=False, greedy=False),
        # An ordinary serving batch with full drafts (all positions in one row pass).
        dict(name="c3_serving", op="verify", recipe="c3", batch=64, k_max=8, vocab=151936, dtype="bf16",
             ragged=False, greedy=False),
        # The headline: a large ragged batch, long drafts, two row windows.
        dict(name="c4_large_ragged", op="verify", recipe="c4", batch=256, k_max=16, vocab=128256, dtype="bf16",
             ragged=True, greedy=False),
        # The largest call: more sequences than compute units, the largest vocabulary, most drafts rejected early.
        dict(name="c5_largest", op="verify", recipe="c5", batch=512, k_max=8, vocab=256000, dtype="bf16",
             ragged=False, greedy=False),
        # Greedy decoding (the paper's own experiments) on fp32 logits, ragged.
        dict(name="greedy_f32", op="verify", recipe="c4", batch=32, k_max=8, vocab=128256, dtype="f32", ragged=True,
             greedy=True),
        # An odd vocabulary with dense rows: no row but the first starts on a 16-byte boundary.
        dict(name="odd_vocab", op="verify", recipe="c4", batch=256, k_max=8, vocab=50257, dtype="bf16", ragged=True,
             greedy=False),
        # A caller that logs: per-position log-probs and the whole recovery row beside the token.
        dict(name="with_logprobs", op="logprobs", recipe="c3", batch=16, k_max=8, vocab=151936, dtype="bf16",
             ragged=False, greedy=False),
        # Always-on steering of every row of the headline batch (the per-token fusion baseline).
        dict(name="steer_4352", op="steer", recipe="c4", batch=4352, vocab=128256, dtype="bf16", greedy=False),
        # One drafting step of the serving batch: one plain softmax draw per sequence.
        dict(name="draft_step_64", op="sample", recipe="c3", batch=64, vocab=151936, dtype="bf16", greedy=False),
        # The deployment split at the headline batch: top-32 downlink, then the edge's resampling.
        dict(name="split_256", op="split", recipe="c4", batch=256, k_max=3, vocab=128256, dtype="bf16", topk=32,
             greedy=False),
        # The same for a few users on fp32 logits and an odd vocabulary.
        dict(name="split_4_f32", op="split", recipe="c1", batch=4, k_max=4, vocab=50257, dtype="f32", topk=32,
             greedy=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        op = rng.choice(["verify"] * 6 + ["logprobs", "steer", "sample", "split"])
        recipe = rng.choice(sorted(WORKLOADS))
        case = dict(op=op, recipe=recipe, vocab=_log_int(rng, 32000, 256000),
                    dtype="f32" if rng.random() < 0.25 else "bf16", greedy=rng.random() < 0.25)
        if rng.random() < 0.5:
            case["vocab"] &= ~63  # model heads are usually padded; the others stay odd or even as they fall
        if op in ("steer", "sample"):
            case["batch"] = _log_int(rng, 1, MAX_ROWS)
        else:
            case["batch"] = _log_int(rng, 1, 64 if op == "logprobs" else 512)
            case["k_max"] = _log_int(rng, 1, 16) if op != "split" else rng.randint(0, 4)
            if op == "split":
                case["topk"] = rng.choice([8, 16, 32, 64])
            else:
                case["ragged"] = rng.random() < 0.5
        rows = case["batch"] * (case.get("k_max", 0) + 1)
        if 3 * rows * case["vocab"] * _esz(case) > MAX_STATE_BYTES:
            continue
        if work(case)["bytes"] <= max(work(c)["bytes"] for c in listed()):
            return case


def _esz(case):
    return 2 if case["dtype"] == "bf16" else 4


def _shape(case):
    return case["batch"], case.get("k_max", 0)


def prepare(case, seed):
    """Logits, drafts, lengths and uniforms on the GPU, drawn as the repository's input recipe draws them (a
    shared Gaussian part and one of each model's own, a Zipf prior where the recipe has one, drafts from the
    specialist's distribution), and what a serving loop keeps: parameters, workspace and output buffers."""
    w, dev = WORKLOADS[case["recipe"]], torch.device("cuda")
    B, K = _shape(case)
    V = case["vocab"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    prior = None
    if w.zipf:
        prior = -w.zipf * torch.log((torch.randperm(V, generator=gen, device=dev) + 1).float())
    plain = case["op"] == "sample"
    coef = {"S_ctx": w.c_ctx} if plain else {"G": w.c_g, "S_ctx": w.c_ctx, "S_noctx": w.c_noctx}
    s = {k: torch.empty(B, K + 1, V, dtype=dt, device=dev) for k in coef}
    s["draft"] = torch.empty(B, K, dtype=torch.int32, device=dev)
    step = max(1, (64 << 20) // ((K + 1) * V))
    for b0 in range(0, B, step):
        n = min(B, b0 + step) - b0
        z0 = torch.randn(n, K + 1, V, generator=gen, device=dev).mul_(w.sigma)
        if prior is not None:
            z0 += prior
        for k, c in coef.items():
            z = torch.randn(n, K + 1, V, generator=gen, device=dev)
            s[k][b0:b0 + n] = z.mul_(c * w.sigma).add_(z0)
        if K:  # the drafting phase: a draw from softmax(S_ctx / T), by adding Gumbel noise
            e = torch.empty(n, K, V, device=dev).exponential_(generator=gen)
            s["draft"][b0:b0 + n] = (s["S_ctx"][b0:b0 + n, :K].float() / w.temperature - e.log_()).argmax(-1)
    s["uniforms"] = torch.rand(B, K + 1, generator=gen, device=dev)
    s["draft_len"] = None
    if case.get("ragged"):
        s["draft_len"] = torch.randint(1, K + 1, (B,), generator=gen, device=dev, dtype=torch.int32)
    s["case"], s["lam"], s["beta"], s["temperature"] = case, LAMBDA, w.beta, w.temperature
    if case["op"] == "split":  # the row each sequence was rejected at
        s["row"] = torch.randint(0, K + 1, (B,), generator=gen, device=dev, dtype=torch.int32)
        s["u_edge"] = torch.rand(B, generator=gen, device=dev)
    elif case["op"] in ("steer", "sample"):
        for k in coef:
            s[k] = s[k].view(B, V)
    else:
        s["params"] = binding.make_params(B, K, V, dt, lam=LAMBDA, beta=w.beta, temperature=w.temperature,
                                          flags=binding.SS_FLAG_GREEDY if case["greedy"] else 0)
        s["workspace"] = torch.empty(max(256, binding.workspace_bytes(s["params"])), dtype=torch.uint8, device=dev)
        s["accepted_len"] = torch.empty(B, dtype=torch.int32, device=dev)
        s["next_token"] = torch.empty(B, dtype=torch.int32, device=dev)
        s["next_token_logprob"] = torch.empty(B, dtype=torch.float32, device=dev)
    return s


def run(s):
    case = s["case"]
    op, greedy = case["op"], case["greedy"]
    if op == "verify":  # a serving loop's call: buffers kept, device pointers handed over
        binding.verify_block_raw(s["G"], s["S_ctx"], s["S_noctx"], s["draft"], s["draft_len"], s["uniforms"],
                                 s["params"], s["accepted_len"], s["next_token"], s["next_token_logprob"], None, None,
                                 s["workspace"])
        return {k: s[k] for k in ("accepted_len", "next_token", "next_token_logprob")}
    if op == "logprobs":
        return binding.verify_block(s["G"], s["S_ctx"], s["S_noctx"], s["draft"], s["uniforms"], lam=s["lam"],
                                    beta=s["beta"], temperature=s["temperature"], draft_len=s["draft_len"],
                                    want_recovery_logprobs=True, want_draft_logprobs=True,
                                    workspace=s["workspace"], greedy=greedy)
    if op == "steer":
        out = binding.steer_rows(s["G"], s["S_ctx"], s["S_noctx"], s["uniforms"], beta=s["beta"],
                                 temperature=s["temperature"], greedy=greedy)
        return {k: out[k] for k in ("token", "token_logprob")}
    if op == "sample":
        out = binding.sample_rows(s["S_ctx"], s["uniforms"], temperature=s["temperature"], greedy=greedy)
        return {k: out[k] for k in ("token", "token_logprob")}
    index, value = binding.cloud_topk(s["G"], s["S_noctx"], s["row"], beta=s["beta"], topk=case["topk"])
    out = binding.edge_resample(index, value, s["S_ctx"], s["row"], s["u_edge"], beta=s["beta"],
                                temperature=s["temperature"], greedy=greedy)
    return {"index": index, "value": value, **out}


def _tested(case):
    """Expected positions of a sequence that Algorithm 1 tests, and the chance that all of them are accepted."""
    a, K = ACCEPT[case["recipe"]], case["k_max"]
    lens = range(1, K + 1) if case["ragged"] else (K,)
    return (sum((1 - a ** k) / (1 - a) for k in lens) / len(lens), sum(a ** k for k in lens) / len(lens),
            sum(lens) / len(lens))


def work(case):
    """Rows that have to be read once (logits of the positions tested, in the two verifying models; the
    specialist's row at the first rejection; all three at a bonus row), and what is written.  About five
    operations a logit: scale, subtract, exponentiate, add, compare."""
    B, _ = _shape(case)
    V, esz, op = case["vocab"], _esz(case), case["op"]
    out = 12.0 * B
    if op in ("verify", "logprobs"):
        tested, bonus, mean_len = _tested(case)
        rows = 2 * (tested if op == "verify" else mean_len) + 1 + 2 * bonus
        if op == "logprobs":
            out += 4.0 * B * V + 8.0 * B * case["k_max"]
    elif op == "split":
        rows = 2.0
        out += 8.0 * B * case["topk"]
    else:
        rows = 3.0 if op == "steer" else 1.0
    return {"bytes": rows * B * V * esz + out, "flops": 5.0 * rows * B * V}


def tolerance(case):
    """Log-probs are stored in fp32 (3e-8 of the value, which is what is measured over a batch) behind fp32
    sums of up to 256000 terms, good to a few 1e-7 in absolute terms.  In a small batch all of them may lie
    close to zero (a peaked row), where that absolute error is a larger share.
    A drawn token differs where a uniform falls on the edge of its interval to within the rounding of the
    cumulative sum; with some 1e5 edges a row that is about one row in 1e4 (seen: one of 4352), and that row's
    log-prob is then another token's.  One such row among N is up to 0.4 / sqrt(N) of the whole."""
    if case["batch"] >= 32 and not case["greedy"] and case["op"] != "split":
        return {"rel": 0.03, "max": 0.99, "differ": 0.004}
    rel = 1e-6 if case["batch"] >= 16 else 1e-4
    return {"rel": rel, "max": 40 * rel, "differ": 0.004}


def _draw_f64(h, temperature, u, greedy):
    """Token and log-prob of softmax(h / T) for rows h [n, V] in double."""
    lp = torch.log_softmax(h / temperature, -1)
    if greedy:
        tok = h.argmax(-1)
    else:
        cdf = torch.cumsum(lp.exp(), -1)
        tok = torch.searchsorted(cdf, u.double()[:, None], right=True)[:, 0].clamp_(max=h.shape[1] - 1)
    return tok, lp, lp.gather(1, tok[:, None])[:, 0]


def exact(case, seed):
    s = prepare(case, seed)
    B, K = _shape(case)
    V, op = case["vocab"], case["op"]
    T, beta = (torch.tensor(s[k], dtype=torch.float32).item() for k in ("temperature", "beta"))  # passed as fp32
    dev = s["uniforms"].device
    step = max(1, (32 << 20) // ((K + 1) * V))
    chunks = [(b0, min(B, b0 + step)) for b0 in range(0, B, step)]
    if op in ("steer", "sample"):
        tok = torch.empty(B, dtype=torch.int32, device=dev)
        tlp = torch.empty(B, dtype=torch.float64, device=dev)
        for b0, b1 in chunks:
            if op == "steer":
                h = s["G"][b0:b1].double() + beta * (s["S_ctx"][b0:b1].double() - s["S_noctx"][b0:b1].double())
            else:
                h = s["S_ctx"][b0:b1].double()
            tok[b0:b1], _, tlp[b0:b1] = _draw_f64(h, T, s["uniforms"][b0:b1, 0], case["greedy"])
        return {"token": tok, "token_logprob": tlp}
    at = torch.arange(B, device=dev)
    if op == "split":
        k = case["topk"]
        index = torch.empty(B, k, dtype=torch.int32, device=dev)
        value = torch.empty(B, k, dtype=torch.float64, device=dev)
        for b0, b1 in chunks:
            r = s["row"][b0:b1].long()
            n = torch.arange(b1 - b0, device=dev)
            h = s["G"][b0:b1][n, r].double() - beta * s["S_noctx"][b0:b1][n, r].double()
            v, i = torch.sort(h, dim=-1, descending=True, stable=True)
            index[b0:b1], value[b0:b1] = i[:, :k], v[:, :k]
        hp = s["S_ctx"][at, s["row"].long()].gather(1, index.long()).double()
        j, _, lp = _draw_f64(value.float().double() + beta * hp, T, s["u_edge"], case["greedy"])
        return {"index": index, "value": value, "next_token": index.gather(1, j[:, None])[:, 0],
                "next_token_logprob": lp}
    lens = torch.full((B,), K, device=dev) if s["draft_len"] is None else s["draft_len"].long()
    lp = torch.empty(B, K, 2, dtype=torch.float64, device=dev)
    for b0, b1 in chunks:
        y = s["draft"][b0:b1].long()[..., None]
        for x, k in enumerate(("G", "S_noctx")):
            z = s[k][b0:b1, :K].double() / T
            lp[b0:b1, :, x] = (z.gather(2, y) - torch.logsumexp(z, -1, keepdim=True))[..., 0]
    t = torch.arange(K, device=dev)
    alpha = torch.exp(lp[..., 0] - lp[..., 1] - math.log(s["lam"])).clamp(max=1.0)
    rejected = (s["uniforms"][:, :K].double() > alpha) & (t < lens[:, None])
    first = torch.where(rejected, t, K + 1).amin(1)
    n = torch.minimum(first, lens)
    tok = torch.empty(B, dtype=torch.int32, device=dev)
    tlp = torch.empty(B, dtype=torch.float64, device=dev)
    rec = torch.empty(B, V, dtype=torch.float64, device=dev) if op == "logprobs" else None
    for b0, b1 in chunks:
        i, r = torch.arange(b1 - b0, device=dev), n[b0:b1]
        g, p, m = (s[k][b0:b1][i, r].double() for k in ("G", "S_ctx", "S_noctx"))
        tok[b0:b1], row, tlp[b0:b1] = _draw_f64(g + beta * (p - m), T, s["uniforms"][b0:b1, K], case["greedy"])
        if rec is not None:
            rec[b0:b1] = row
    out = {"accepted_len": n.int(), "next_token": tok, "next_token_logprob": tlp}
    if op == "logprobs":
        lp[t >= lens[:, None]] = 0.0
        out.update(recovery_logprobs=rec, draft_logprobs=lp)
    return out
