"""Which blocks the static scratch takes does not depend on how the library lays its workspace out (CPU)."""
import random

import torch

from paper_2603_16219_amd import binding as B


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
