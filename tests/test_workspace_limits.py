"""Which blocks the static scratch takes does not depend on how the library lays its workspace out (CPU)."""
import random

import pytest

import torch

from paper_2603_16219_amd import binding as B
from test_plan_host import planner  # noqa: F401  the planner compiled on its own


def up(x):
    return (x + 255) // 256 * 256


def slices(nvec, row_tensors):
    want = -(-32768 // row_tensors) if row_tensors > 0 else 1
    ns = max(1, min(64, max(-(-nvec // 4096), min(-(-nvec // 256), want))))
    sv = -(-(-(-nvec // ns)) // 256) * 256
    return max(1, -(-nvec // sv))


def least_bytes(p):
    """Two row lists, four words a sequence, slice partials of every position at the finest of three slicings
    (one window of all positions, or a quarter of them and the rest),
    and up to 128 sequences a counter, 256 bytes and 8 bytes a recovery chunk each."""
    vec = 8 if p.dtype == B.SS_BF16 else 4
    nvec = -(-p.vocab // vec)
    t1 = p.k_max // 4 if B.first_window(p) < p.k_max else p.k_max
    ns = max(slices(nvec, 2 * p.batch * t1), slices(nvec, 2 * p.batch * (p.k_max - t1) // 3), slices(nvec, 2 * p.batch * p.k_max))
    total = 2 * up(4 * (p.batch + 1)) + 3 * up(4 * max(p.batch, 1)) + up((p.batch * p.k_max * 2 + 1) * ns * 8)
    if 1 <= p.batch <= 128:
        nfull = p.vocab // vec
        nc = -(-nfull // 256) + (1 if p.vocab % vec else 0)
        total += up(4 * p.batch) + up(256 * p.batch) + up(8 * p.batch * nc)
    return total


def test_the_blocks_that_fit_the_static_scratch_are_the_same():
    rng = random.Random(7)
    near = 0
    for _ in range(4000):
        batch = int(2 ** rng.uniform(0, 14))
        k_max = rng.choice([0, 1, 2, 3, 4, 7, 8, 16, 33, 64, 200])
        vocab = int(2 ** rng.uniform(0, 20))
        p = B.make_params(batch, k_max, vocab, rng.choice([torch.bfloat16, torch.float32]), lam=0.5, beta=1.0,
                          temperature=1.0, flags=rng.choice([0, B.SS_FLAG_GREEDY, B.SS_FLAG_FULL_ROWS]))
        got, least = B.workspace_bytes(p), least_bytes(p)
        assert got >= least, (batch, k_max, vocab)
        assert (got <= B.STATIC_SCRATCH_BYTES) == (least <= B.STATIC_SCRATCH_BYTES), (batch, k_max, vocab, got, least)
        near += 0.5 < least / B.STATIC_SCRATCH_BYTES < 2
    assert near > 100


def bytes_without_logits(p):
    """What a block needs if the draft tokens' logits are gathered: least_bytes, and up to 128 sequences the tables of a
    shared recovery row in the place of its last term unless they alone keep the block out of the static scratch."""
    least = least_bytes(p)
    if not 1 <= p.batch <= 128:
        return least
    vec = 8 if p.dtype == B.SS_BF16 else 4
    chunks = lambda v: -(-(v // vec) // 256) + (1 if v % vec else 0)
    nc = max(chunks(p.vocab), chunks(p.vocab + 1)) if vec == 8 else chunks(p.vocab)
    tables = up(256 * p.batch) + up(8 * p.batch * max(nc, 32)) + up(4 * p.batch * nc) + up(8 * p.batch * nc)
    whole = least - up(4 * p.batch) - up(256 * p.batch) - up(8 * p.batch * chunks(p.vocab)) + tables
    return least if least <= B.STATIC_SCRATCH_BYTES < whole else whole


def test_a_workspace_without_space_for_the_draft_logits_will_do(planner):  # noqa: F811
    """Beyond 512 draft positions; up to them the block lies so far below the static scratch's limit that it never asks for less
    than a smaller one because of them."""
    rng = random.Random(8)
    asked, want = [], []
    for i in range(6000):
        batch = int(2 ** rng.uniform(0, 14))
        k_max = rng.choice([0, 1, 2, 4, 8, 16, 64, 200, 1000])
        vocab = int(2 ** rng.uniform(0, 20))
        dt = rng.choice([torch.bfloat16, torch.float32])
        if (batch + 1) * (k_max + 1) > 1 << 30:
            continue
        p = B.make_params(batch, k_max, vocab, dt, lam=0.5, beta=1.0, temperature=1.0)
        need, lean = B.workspace_bytes(p), bytes_without_logits(p)
        assert need in (lean, lean + up(8 * batch * k_max)), (batch, k_max, vocab)
        if batch * k_max <= 512:
            assert need == lean + up(8 * batch * k_max) < B.STATIC_SCRATCH_BYTES or need == lean > B.STATIC_SCRATCH_BYTES
        least = lean if batch * k_max > 512 else need
        for n in (need, least, least - 1, least - 256):
            asked.append(f"within {batch} {k_max} {vocab} {p.dtype} 0 0.5 {n}")
            want.append((1, 1 if n >= lean + up(8 * batch * k_max) else 0) if n >= least else (0,))
    for line, g, x in zip(asked, planner(asked), want):
        assert g[:len(x)] == x, (line, g, x)


@pytest.mark.parametrize("more,fewer,k_max,vocab", [(350, 349, 1000, 40), (1741, 1740, 200, 40), (5391, 5390, 64, 40)])
def test_the_workspace_of_a_larger_batch_will_do(planner, more, fewer, k_max, vocab):  # noqa: F811
    """Where only a plan without the draft tokens' logits fits the static scratch the larger batch asks for less."""
    p = [B.make_params(b, k_max, vocab, torch.bfloat16, lam=0.5, beta=1.0, temperature=1.0) for b in (more, fewer)]
    held, need = (B.workspace_bytes(x) for x in p)
    assert bytes_without_logits(p[1]) <= held
    assert planner([f"within {fewer} {k_max} {vocab} {B.SS_BF16} 0 0.5 {held}"])[0][0] == 1
