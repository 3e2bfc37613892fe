"""GPU parity of the bf16 attention kernels for head dim 64 beyond 128 rows per kv-head.

Blocks of up to 192 rows on eight waves of two 16-row groups or on four of three, and
blocks of up to 256 rows on eight waves of 32 rows: row counts around the groups and
blocks of all, sequences with fewer nodes than the launch, against the float64 oracle
on sampled nodes.
"""

import math

import pytest
import torch

import paper_2608_00531_amd as pc
from test_gpu_tree_attn_general import general_tree_workload
from parity_util import say, upload, gpu_attn, oracle_attn, check_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,group,nodes,ctx", [
    # up to 256 workgroups: eight waves of row groups, blocks of up to 192 rows
    (2, 1, [129, 144], [300, 64]), (1, 8, [17, 18], [700, 90]), (2, 4, [64, 33], [129, 1000]),
    (1, 4, [65, 20], [500, 500]), (1, 8, [100, 256], [10, 70]),
    # more workgroups: four waves, and eight of 32 rows (200, 240, 256 and 2048 rows)
    (8, 4, [33, 48], [13000, 12800]), (8, 4, [48, 48], [25700, 0]), (4, 8, [25, 40], [14000, 13000]),
    (2, 8, [256, 199], [13000, 500]), (8, 4, [60, 49], [26000, 100])])
@pytest.mark.parametrize("kv_split", [0, 3])
def test_row_groups_and_blocks(hkv, group, nodes, ctx, kv_split):
    say("d64", hkv, group, nodes, ctx, kv_split)
    w = general_tree_workload(31, 2, hkv, group, 64, nodes, ctx, "nested")
    sample = [(b, i) for b in (0, 1) for i in sorted({0, nodes[b] // 2, nodes[b] - 2, nodes[b] - 1}) if i >= 0]
    o, lse, st = gpu_attn(w, upload(w), kv_split=kv_split)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * 2
    check_attn(w, o, lse, *oracle_attn(w, sample=sample), sample=sample)


@pytest.mark.parametrize("batch", [2, 40])             # up to 32 workgroups, and 320 or more
@pytest.mark.parametrize("nodes", [33, 48, 64])        # one block of 132, 192 and 256 rows (or two of 128)
def test_probabilities_are_rounded_against_the_first_64_tokens(batch, nodes):
    """The output in fp32 against float64 sums of probabilities that are rounded to bf16 relative to
    each row's maximum over the split's first 64 tokens. A kernel's fp32 scores (relative error about
    5e-7) move one probability in 4000 across a rounding boundary, by 2^-8: 6e-5 of the output; the
    maximum of another set of tokens moves nearly all (2e-3)."""
    say("d64 reference", batch, nodes)
    hq, hkv, d, ctx, scale = 32, 8, 64, 230, 0.125
    gen = torch.Generator(device="cuda").manual_seed(nodes)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda").bfloat16()
    rows = ctx + nodes
    q, k, v = draw(batch, nodes, hq, d), draw(batch * rows, hkv, d), draw(batch * rows, hkv, d)
    i32 = dict(dtype=torch.int32, device="cuda")
    o, lse, st = pc.cure_tree_attn(
        q, k, v, torch.arange(batch, device="cuda") * rows, torch.full((batch,), ctx, **i32),
        torch.full((batch,), nodes, **i32), torch.arange(-1, nodes - 1, **i32).repeat(batch, 1),
        [ctx] * batch, [nodes] * batch, scale, out_dtype=torch.float32, kv_split=1)
    torch.cuda.synchronize()
    hidden = torch.ones(nodes, nodes, dtype=torch.bool, device="cuda").triu(1)      # the tree is a chain
    for b in (0, batch - 1):
        for h in range(hq):
            kb, vb = (t[b * rows:(b + 1) * rows, h * hkv // hq].double() for t in (k, v))
            x = q[b, :, h].double() @ kb.t().contiguous() * (scale / math.log(2.0))
            x[:, ctx:].masked_fill_(hidden, -math.inf)
            p = torch.exp2(x - x[:, :64].amax(dim=1, keepdim=True)).float().bfloat16().double()
            want = p @ vb / p.sum(dim=1, keepdim=True)
            assert float((o[b, :, h].double() - want).norm() / want.norm()) < 3e-4, (b, h)
