"""GPU parity of the fp32 matrix-core attention kernel at the edges of its dispatch.

The kernel works on blocks of 32 query rows (16 when a kv-head has no more), its four
waves over the block's 16-row groups and two or four shares of each tile's tokens, and
takes operands that are 16-byte aligned; everything else in fp32 stays on the
vector-ALU kernel.
Outputs against the float64 oracle at the fp32 bars of the other fp32 tests
(1e-5 output, 1e-4 log-sum-exp: sums of a few hundred fp32 terms of N(0, 1)
inputs, each rounded at 2^-24).
"""

import numpy as np
import pytest
import torch

import paper_2608_00531_amd as pc
from test_gpu_tree_attn_general import general_tree_workload
from parity_util import say, upload, gpu_attn, oracle_attn, check_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hkv,group,nodes", [
    (2, 1, [1, 3]), (2, 1, [16, 9]), (1, 4, [4, 2]),       # up to 16 rows: tokens over 4 waves
    (2, 1, [17, 32]), (3, 2, [16, 5]),                     # up to 32 rows: tokens over 2 waves
    (2, 1, [33, 8]), (2, 4, [16, 15]), (1, 8, [9, 80])])   # row blocks of 32
@pytest.mark.parametrize("ctx,kv_split", [([0, 31], 0), ([63, 130], 0), ([500, 1], 3), ([257, 640], 0)])
def test_row_and_token_shares(d, hkv, group, nodes, ctx, kv_split):
    say("f32", d, hkv, group, nodes, ctx, kv_split)
    w = general_tree_workload(5, 2, hkv, group, d, nodes, ctx, "nested", dtype="f32")
    o, lse, st = gpu_attn(w, upload(w), kv_split=kv_split)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * 2
    check_attn(w, o, lse, *oracle_attn(w))


@pytest.mark.parametrize("nodes,ctx", [
    ([80] * 8, [1400] * 8), ([80, 80, 31, 80, 80, 0, 80, 64], [1400, 400, 650, 100, 1300, 0, 1000, 300])])
def test_splits_of_launches_that_overfill_the_chip(nodes, ctx):
    """640 blocks of 32 rows, as single splits 62 % of the two rounds that they take on 256 CUs, run in
    shorter splits instead."""
    say("f32 tail", nodes, ctx)
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    blocks = 8 * 8 * (80 * 4 // 32)
    assert blocks > slots and 5 * blocks < 4 * (-(-blocks // slots) * slots)
    w = general_tree_workload(10, 8, 8, 4, 128, nodes, ctx, "nested", dtype="f32")
    sample = [(b, i) for b in range(8) for i in sorted({0, nodes[b] // 2, nodes[b] - 1}) if 0 <= i < nodes[b]]
    o, lse, st = gpu_attn(w, upload(w))
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * 8
    check_attn(w, o, lse, *oracle_attn(w, sample=sample), sample=sample)


@pytest.mark.parametrize("scale", [-0.125, 0.0])
def test_nonpositive_scale(scale):
    say("f32 scale", scale)
    w = general_tree_workload(6, 2, 2, 4, 128, [12, 7], [150, 40], "forest", dtype="f32")
    w.scale = scale
    o, lse, _ = gpu_attn(w, upload(w))
    torch.cuda.synchronize()
    check_attn(w, o, lse, *oracle_attn(w))


def test_unaligned_operands_and_bf16_output():
    """Tensors that start between 16-byte boundaries are taken as before, and a bf16 output is the
    rounded fp32 one (half an ulp of bf16 plus the fp32 bar)."""
    w = general_tree_workload(7, 2, 2, 4, 64, [12, 7], [150, 40], "forest", dtype="f32")
    dev = upload(w)
    ref_o, ref_l = oracle_attn(w)
    for name in ("q", "k", "v"):
        t = torch.empty(dev[name].numel() + 1, device="cuda")[1:].view(dev[name].shape)
        moved = dict(dev, **{name: t.copy_(dev[name])})
        assert moved[name].data_ptr() % 16 == 4
        o, lse, _ = gpu_attn(w, moved)
        torch.cuda.synchronize()
        check_attn(w, o, lse, ref_o, ref_l)
    o, _, _ = gpu_attn(w, dev, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for b in range(2):
        n = int(w.n_nodes[b])
        err = np.abs(o[b, :n].float().cpu().numpy() - ref_o[b, :n])
        assert np.all(err <= np.abs(ref_o[b, :n]) * 2.0 ** -8 + 1e-5)


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("group", [1, 2, 8])
def test_hidden_keys_leave_the_other_nodes_alone(value, group):
    """An infinite or NaN key of one node reaches only that node and its descendants."""
    w = general_tree_workload(8, 1, 2, group, 64, [14], [100], "uniform", dtype="f32")
    parent = w.parent[0]
    bad = 5
    sees = np.zeros(14, bool)
    for i in range(14):
        sees[i] = i == bad or (parent[i] >= 0 and sees[parent[i]])
    ref_o, ref_l = oracle_attn(w)
    w.k[100 + bad] = value
    o, lse, st = gpu_attn(w, upload(w))
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK]
    check_attn(w, o, lse, ref_o, ref_l, sample=[(0, i) for i in range(14) if not sees[i]])


def test_malformed_tree_status():
    w = general_tree_workload(9, 3, 2, 1, 64, [10, 20, 12], [70, 10, 300], "nested", dtype="f32")
    w.parent[1, 4] = 9
    dev = upload(w)
    o, lse, st = gpu_attn(w, dev)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK, pc.CURE_ERR_BAD_TREE, pc.CURE_OK]
    w.parent[1, 4] = 3
    ref_o, ref_l = oracle_attn(w)
    check_attn(w, o, lse, ref_o, ref_l, sample=[(b, n) for b in (0, 2) for n in range(int(w.n_nodes[b]))])


@pytest.mark.parametrize("host", [300, 140000])
def test_sequences_beyond_32_bit_offsets(host):
    """A sequence whose K rows take more than 4 GiB, known to the host or not: sampled heads against
    float64 sums (fp32 bars; 4.6 GB each of K and V)."""
    say("f32 long", host)
    ctx, n, h, d = 140000, 3, 64, 128
    gen = torch.Generator(device="cuda").manual_seed(11)
    draw = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    q, k, v = draw(1, n, h, d), draw(ctx + n, h, d), draw(ctx + n, h, d)
    i32 = dict(dtype=torch.int32, device="cuda")
    o, lse, st = pc.cure_tree_attn(q, k, v, torch.zeros(1, dtype=torch.int64, device="cuda"),
                                   torch.tensor([ctx], **i32), torch.tensor([n], **i32),
                                   torch.tensor([[-1, 0, 1]], **i32), [host], [n], 0.125)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK]
    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    for i in (0, 31, 63):
        x = q[0, :, i].double() @ k[:, i].double().t().contiguous() * 0.125
        x[:, ctx:].masked_fill_(hidden, -float("inf"))
        want = torch.softmax(x, dim=1) @ v[:, i].double()
        assert float((o[0, :, i].double() - want).abs().max()) <= 1e-5
        assert float((lse[0, :, i].double() - torch.logsumexp(x, dim=1)).abs().max()) <= 1e-4
