"""GPU parity of ragged attention launches, which may hold only the workgroups with work.

The host lists each sequence's splits in the kernel arguments (up to 64 sequences
and 512 splits in all, where a grid over sequences and splits would not fit the GPU
at one workgroup per CU); other launches are that grid. Both
forms against the float64 oracle: at the limits of the list, with sequences
without nodes or context, with forced split counts, for every kernel family, and
with host sizes that are not the device's (they only plan the launch, so any
nonnegative ones within n_max have to give the same result).
"""

import numpy as np
import pytest
import torch

import paper_2608_00531_amd as pc
from test_gpu_tree_attn_general import general_tree_workload
from parity_util import say, upload, gpu_attn, oracle_attn, check_attn

pytestmark = pytest.mark.gpu


def check(w, dev, ref, **kw):
    o, lse, st = gpu_attn(w, dev, **kw)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * w.batch
    check_attn(w, o, lse, *ref)


@pytest.mark.parametrize("dtype,hkv,group,d,nodes", [
    ("bf16", 2, 4, 128, [16, 9, 0, 16, 3]), ("bf16", 1, 4, 128, [48, 40, 48, 0, 33]),
    ("bf16", 1, 4, 128, [80, 80, 65, 10, 0]), ("bf16", 2, 4, 128, [120, 4, 0, 100, 77]),
    ("bf16", 3, 2, 64, [20, 0, 7, 20, 20]), ("bf16", 1, 4, 64, [48, 30, 48, 0, 11]),
    ("bf16", 1, 4, 64, [60, 49, 60, 0, 11]),
    ("f32", 2, 4, 64, [12, 0, 12, 5, 1]), ("f32", 1, 1, 128, [9, 16, 2, 0, 16])])
@pytest.mark.parametrize("kv_split", [0, 5])
@pytest.mark.parametrize("heads", ["few", "many"])
def test_every_kernel_family(dtype, hkv, group, d, nodes, kv_split, heads):
    say("ragged", dtype, hkv, group, d, nodes, kv_split, heads)
    ctx, sample = [700, 0, 300, 1500, 65], None
    if heads == "many":                       # five splits or more of five sequences, 14 heads: listed
        hkv, sample = 14, [(b, i) for b in range(5) for i in sorted({0, nodes[b] // 2, nodes[b] - 1}) if 0 <= i < nodes[b]]
    w = general_tree_workload(21, 5, hkv, group, d, nodes, ctx, "nested", dtype=dtype)
    o, lse, st = gpu_attn(w, upload(w), kv_split=kv_split)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * 5
    check_attn(w, o, lse, *oracle_attn(w, sample=sample), sample=sample)


@pytest.mark.parametrize("batch", [63, 64, 65])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_batches_around_the_list_of_sequences(batch, dtype):
    rng = np.random.default_rng(batch)
    ctx = [int(c) for c in rng.integers(0, 900, batch)]
    nodes = [int(n) for n in rng.integers(0, 9, batch)]
    nodes[-1], ctx[-1] = 8, 899
    w = general_tree_workload(22, batch, 3, 4, 64, nodes, ctx, "uniform", dtype=dtype)
    check(w, upload(w), oracle_attn(w))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("last,listed", [(61, 511), (62, 512), (63, 513)])
def test_splits_around_the_list(last, listed, dtype):
    """The list holds 512 splits: one less, as many and one more. Sequences that take 64-token splits,
    the longest one 200 of them, with some tokens in each one's last."""
    splits, nodes = [200, 150, 100, last], [6, 6, 3, 6]
    ctx = [64 * s - 30 - n for s, n in zip(splits, nodes)]
    assert sum(-(-(c + n) // 64) for c, n in zip(ctx, nodes)) == listed
    w = general_tree_workload(23, 4, 1, 2, 64, nodes, ctx, "uniform", dtype=dtype)
    check(w, upload(w), oracle_attn(w), kv_split=200)


@pytest.mark.parametrize("dtype,group", [("bf16", 4), ("f32", 2)])
@pytest.mark.parametrize("host", ["larger", "smaller", "swapped", "none_here"])
@pytest.mark.parametrize("hkv", [2, 24])               # a full grid, and listed (but for "smaller")
def test_host_sizes_only_plan(dtype, group, host, hkv):
    ctx, nodes = [700, 300, 1500, 65], [16, 12, 16, 5]
    w = general_tree_workload(24, 4, hkv, group, 128, nodes, ctx, "forest", dtype=dtype)
    dev, ref = upload(w), oracle_attn(w)
    hc, hn = {"larger": ([2000, 900, 1600, 900], [16] * 4), "smaller": ([300, 20, 700, 0], [3, 1, 16, 5]),
              "swapped": (ctx[::-1], nodes[::-1]), "none_here": ([700, 300, 1500, 65], [0, 12, 16, 0])}[host]
    o, lse, st = pc.cure_tree_attn(dev["q"], dev["k"], dev["v"], dev["kv_off"], dev["ctx_len"], dev["n_nodes"],
                                   dev["parent"], hc, hn, w.scale)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * 4
    check_attn(w, o, lse, *ref)


@pytest.mark.parametrize("d,hkv,group,kv_split", [(128, 8, 4, 2), (128, 8, 4, 4), (128, 8, 4, 5), (64, 8, 4, 3),
                                                  (64, 3, 7, 2), (128, 3, 7, 3)])
@pytest.mark.parametrize("ragged", [False, True])
def test_merges_of_many_rows(d, hkv, group, kv_split, ragged):
    """Launches of at least 16384 output rows and up to four splits take the merge with several rows
    to a wave; head counts that its workgroups do not divide, stale slots and lone splits among them."""
    batch, n = 26, 32
    ctx = [(290 - 9 * i if ragged else 250) for i in range(batch)]
    nodes = [n - (i % 3 if ragged else 0) for i in range(batch)]
    nodes[0] = n
    assert batch * n * hkv * group >= 16384
    w = general_tree_workload(25, batch, hkv, group, d, nodes, ctx, "nested")
    sample = [(b, i) for b in (0, 1, 12, 24, 25) for i in (0, 5, nodes[b] - 1)]
    dev = upload(w)
    pc.cure_tree_attn(dev["q"] * 100, dev["k"], dev["v"], dev["kv_off"], dev["ctx_len"], dev["n_nodes"],
                      dev["parent"], w.ctx_len, w.n_nodes, w.scale, kv_split=9)      # other data in the slots
    o, lse, st = gpu_attn(w, dev, kv_split=kv_split)
    torch.cuda.synchronize()
    assert st.tolist() == [pc.CURE_OK] * batch
    check_attn(w, o, lse, *oracle_attn(w, sample=sample), sample=sample)


@pytest.mark.parametrize("dtype,group,d", [("bf16", 4, 128), ("bf16", 12, 64), ("f32", 2, 128)])
@pytest.mark.parametrize("host", ["swapped", "shorter"])
@pytest.mark.parametrize("hkv", [2, 12])               # a full grid, and listed
def test_a_captured_launch_replays_with_other_lengths(dtype, group, d, host, hkv):
    ctx, nodes = [1500, 300, 2600, 65], [16, 12, 16, 5]
    w = general_tree_workload(26, 4, hkv, group, d, nodes, ctx, "forest", dtype=dtype)
    dev, ref = upload(w), oracle_attn(w)
    hc, hn = (ctx[::-1], nodes[::-1]) if host == "swapped" else ([40, 0, 1900, 65], [1, 0, 16, 5])
    call = lambda: pc.cure_tree_attn(dev["q"], dev["k"], dev["v"], dev["kv_off"], dev["ctx_len"], dev["n_nodes"],
                                     dev["parent"], hc, hn, w.scale)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        call()
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            o, lse, st = call()
        for _ in range(3):
            call()
            o.zero_(), lse.zero_()
            graph.replay()
            stream.synchronize()
            assert st.tolist() == [pc.CURE_OK] * 4
            check_attn(w, o, lse, *ref)
