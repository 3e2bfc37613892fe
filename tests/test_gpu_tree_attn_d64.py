"""GPU parity of the bf16 attention kernels for head dim 64 beyond 128 rows per kv-head.

Blocks of up to 256 rows on waves of two 16-row groups, or, with many tokens per
CU, of up to 192 rows on waves of three: row counts around the groups and blocks
of both, sequences with fewer nodes than the launch, against the float64 oracle
on sampled nodes.
"""

import pytest
import torch

import paper_2608_00531_amd as pc
from test_gpu_tree_attn_general import general_tree_workload
from parity_util import say, upload, gpu_attn, oracle_attn, check_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,group,nodes,ctx", [
    # few tokens per CU: 129 - 256 rows in one block, then two and more
    (2, 1, [129, 144], [300, 64]), (1, 8, [17, 18], [700, 90]), (2, 4, [64, 33], [129, 1000]),
    (1, 4, [65, 20], [500, 500]), (1, 8, [100, 256], [10, 70]),
    # many tokens per CU (at least 204800 tokens x kv-heads x 256-row blocks)
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
