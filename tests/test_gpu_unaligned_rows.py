"""GPU parity of the margin pass and the repair tree on rows that start anywhere.

A row length or a base address that is no multiple of 16 bytes puts each row's
first 16-byte boundary at another entry. The vectors start there; the entries
before and after them are taken singly, as are all of a margin pass's rows of fewer
than 1280 entries. Every base offset of a 16-byte window,
vocabularies around the vector, chunk and loop-step sizes, with the best
entries in the first and last positions of the row and at the chunk edges,
against the oracle: indices bit-exact.
"""

import numpy as np
import pytest
import torch

import oracle
import paper_2608_00531_amd as pc
from synth import make_draft_block
from synth.workloads import bf16_round
from parity_util import say, MARGIN_TOL
from test_gpu_repair import run_case

pytestmark = pytest.mark.gpu


def shifted(a, dtype, off):
    """`a` on the GPU, its first element `off` elements past a 16-byte boundary."""
    t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16 if dtype == "bf16" else np.float32))
    buf = torch.zeros(t.numel() + 16, dtype=t.dtype, device="cuda")
    assert buf.data_ptr() % 16 == 0
    x = buf[off:off + t.numel()].view(a.shape).copy_(t)
    return x.view(torch.bfloat16) if dtype == "bf16" else x


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab", [2, 5, 9, 17, 1279, 1280, 1289, 8191, 8200, 16385, 50257, 70001])
def test_margins_on_rows_that_start_anywhere(dtype, vocab):
    rng = np.random.default_rng(vocab)
    rows = 24
    x = rng.standard_normal((rows, vocab)).astype(np.float32)
    edges = [0, 1, 6, 7, 8, 9, vocab // 2, vocab - 9, vocab - 8, vocab - 2, vocab - 1]
    for r in range(rows - 4):                       # the last rows keep the noise's own order
        i, j = rng.choice([e for e in edges if 0 <= e < vocab], 2)
        x[r, i] = 8.0
        x[r, j] = 8.0 if r % 3 == 0 else 9.0       # ties too
    x[0, :] = -np.inf
    x[0, vocab - 1] = 1.0
    bits = bf16_round(x) if dtype == "bf16" else x
    if dtype == "bf16":
        bits[0, :vocab - 1] = 0xff80                # -inf (the rounding helper takes finite values)
    ref = oracle.margins(bits, dtype)
    for off in range(8 if dtype == "bf16" else 4):
        say("margins", dtype, vocab, "offset", off)
        got = pc.cure_margins(shifted(bits[None], dtype, off), chain_len=rows, repair_budget=8)
        torch.cuda.synchronize()
        for k in ("top1_idx", "top2_idx", "top1_val", "top2_val"):
            assert np.array_equal(got[k][0].cpu().numpy(), ref[k]), (k, off)
        err = np.abs(got["lse"][0].cpu().numpy() - ref["lse"])
        assert np.max(err) <= MARGIN_TOL


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vocab", [9, 16, 23, 8192, 8193, 8199, 16384, 32001])
def test_repair_trees_on_rows_that_start_anywhere(dtype, vocab):
    blk = make_draft_block(batch=2, chain_len=6, vocab=vocab, dtype=dtype, seed=vocab % 89, n_low=4,
                           runners=min(6, vocab - 1), depth=2)
    if vocab > 100:                                 # equal values beyond a wave's list: the long way round
        blk.logits[0, 2, :300] = blk.logits[0, 2].max() if dtype == "f32" else bf16_round(
            np.float32([40.0]))[0]
    for off in range(8 if dtype == "bf16" else 4):
        say("repair", dtype, vocab, "offset", off)
        run_case(blk, tau=1.5, budget=16, depth=2, scale=1.0, b_min=1, b_max=5,
                 logits_dev=shifted(blk.logits, dtype, off))


@pytest.mark.parametrize("dtype,off", [("bf16", 1), ("bf16", 5), ("f32", 1), ("f32", 3)])
def test_a_nan_beside_the_vectors_hides_no_other_entry(dtype, off):
    """The ranking passes over a NaN: one among a row's first or last entries leaves the tree as if it
    were -inf, also where many equal values send a wave the long way round."""
    say("repair nan", dtype, off)
    vocab, head = 8203, (8 if dtype == "bf16" else 4) - off
    trees = []
    for value in (np.nan, -np.inf):
        x = np.full((1, 1, vocab), -4.0, np.float32)
        x[0, 0, 600:1000] = 2.0
        x[0, 0, head:head + 3] = [9.0, 8.0, 7.0]              # in the first lane's vector, like the NaN's lane
        x[0, 0, [0, vocab - 1]] = value
        t = torch.from_numpy(x).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        buf = torch.zeros(vocab + 16, dtype=t.dtype, device="cuda")
        row = buf[off:off + vocab].view(1, 1, vocab).copy_(t)
        i32 = dict(dtype=torch.int32, device="cuda")
        trees.append(pc.cure_repair_tree(row, torch.zeros(1, 1, device="cuda"), torch.zeros(1, 1, **i32),
                                         torch.ones(1, **i32), torch.full((1, 1), 5000, **i32), 5, 1, 1.0,
                                         b_min=5, b_max=5))
    assert trees[0]["token"][0].tolist() == [5000, head, head + 1, head + 2, 600, 601]
    assert all(torch.equal(trees[0][k], trees[1][k]) for k in trees[0])
