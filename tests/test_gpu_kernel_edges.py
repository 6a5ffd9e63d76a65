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


# The log-prob rows are cut into segments of 512 vectors (4096 bf16 or 2048 fp32 logits): one segment exactly,
# one logit more and less, a last segment that holds only the logits past the last vector, less than a vector.
@pytest.mark.parametrize("beta", [0.0, 0.8])
@pytest.mark.parametrize("dtype,vocab", [("bf16", 4096), ("bf16", 4097), ("bf16", 8191), ("bf16", 3), ("f32", 2048),
                                         ("f32", 2049), ("f32", 6143), ("f32", 3)])
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
