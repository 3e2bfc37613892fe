"""Which kernels a call launches, and with how many workgroups, on the CPU.

A stub of the HIP runtime (launch_stub.cpp) records the launches of the built library in a
process of its own; nothing runs on a GPU.
"""

import json
import os
import subprocess
import sys

import pytest

from paper_2608_00531_amd import build as pbuild

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import ctypes as c, json, sys
stub = c.CDLL(sys.argv[1], c.RTLD_GLOBAL)            # before the library's own HIP runtime
stub.stub_launches.restype = c.c_char_p
lib = c.CDLL(sys.argv[2])
p, i, f, z = c.c_void_p, c.c_int32, c.c_float, c.c_size_t
attn = lib.cure_tree_attn
attn.argtypes = [p] * 5 + [i] * 6 + [f] + [p] * 4 + [i, p, p, i, c.c_uint32, p, p, z, p]
lib.cure_margins.argtypes = [p, i, i, i, i, c.c_int64] + [p] * 6 + [i, f, i, i, p, p, p, z, p]
def margins(vocab, ld, offset, dtype):
    stub.stub_reset(0)
    t = 4096
    status = lib.cure_margins(t + offset, 0 if dtype == "f32" else 1, 1, 4, vocab, ld, t, t, t, t, t, t, 0, 1.0, 0, 1,
                              None, None, t, 1 << 60, None)
    return status, [l.split() for l in stub.stub_launches().decode().splitlines()]
def attention(ctx, nodes, hq, hkv, d, dtype="bf16", kv_split=0, capturing=False):
    array = lambda v: (i * len(v))(*v)
    t, b = 4096, len(ctx)
    stub.stub_reset(int(capturing))
    code = 0 if dtype == "f32" else 1
    status = attn(t, t, t, t, t, code, code, b, hq, hkv, d, 0.125, t, t, t, t, max(nodes), array(ctx),
                  array(nodes), kv_split, 0, t, t, 1 << 60, None)
    return status, [l.split() for l in stub.stub_launches().decode().splitlines()]
print(json.dumps([(margins if "vocab" in kw else attention)(**kw) for kw in json.loads(sys.argv[3])]))
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    stub = str(tmp_path_factory.mktemp("stub") / "launch_stub.so")
    res = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(HERE, "launch_stub.cpp"),
                          "-o", stub], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def run(*calls):
        """Per call: its kernels as (mangled name, grid, threads per workgroup)."""
        res = subprocess.run([sys.executable, "-c", CHILD, stub, pbuild.LIB_PATH, json.dumps(calls)],
                             capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stdout + res.stderr
        out = json.loads(res.stdout)
        assert all(status == 0 for status, _ in out), out
        return [[(l[0], tuple(map(int, l[1:4])), int(l[4])) for l in got] for _, got in out]
    return run


def is_compact(launch):
    return "CompactArgs" in launch[0]


# Eight sequences of 100 to 4000 tokens and 32 nodes, 8 kv-heads: forced splits of 512 tokens.
RAGGED = dict(ctx=[4000, 100, 900, 1500, 2000, 300, 3000, 600], nodes=[32] * 8, hq=32, hkv=8, d=128, kv_split=8)
SPLITS = [-(-(c + 32) // 512) for c in RAGGED["ctx"]]


def test_a_captured_ragged_launch_has_room_for_other_lengths(launches):
    """A launch that is replayed may meet a sequence that has grown since: each one has the launch's
    largest split count at its disposal, where a call that runs once holds only the splits in use."""
    eager, captured = launches(RAGGED, dict(RAGGED, capturing=True))
    assert max(SPLITS) == 8 and sum(SPLITS) < 64
    assert is_compact(eager[0]) and eager[0][1] == (sum(SPLITS) * 8, 1, 1)
    assert is_compact(captured[0]) and captured[0][1] == (8 * 8 * 8, 1, 1)
    # More than the table holds: the grid over sequences and splits.
    many = dict(RAGGED, ctx=RAGGED["ctx"] * 3, nodes=[32] * 24, kv_split=32)
    eager, captured = launches(many, dict(many, capturing=True))
    assert is_compact(eager[0])
    assert not is_compact(captured[0]) and captured[0][1] == (8, 32, 24)


def test_the_list_holds_512_splits(launches):
    """Sequences of 200, 150, 100 and 61 to 63 splits of 64 tokens: listed up to 512 in all, a grid over
    sequences and splits beyond."""
    call = lambda last: dict(ctx=[64 * s - 36 for s in (200, 150, 100, last)], nodes=[6] * 4, hq=2, hkv=1, d=64,
                             kv_split=200)
    below, at, above = [got[0] for got in launches(call(61), call(62), call(63))]
    assert is_compact(below) and below[1] == (511, 1, 1)
    assert is_compact(at) and at[1] == (512, 1, 1)
    assert not is_compact(above) and above[1] == (1, 200, 4)


def test_grids_stay_below_the_runtimes_limit_of_threads(launches):
    """The runtime takes fewer than 2^32 threads in each grid dimension. 443 splits on 32768 kv-heads are
    14.5 million workgroups of 512 threads: a grid over sequences and splits."""
    call = dict(ctx=[384] * 63 + [64], nodes=[16] * 64, hq=32768, hkv=32768, d=64, kv_split=7)
    few = dict(call, hq=8192, hkv=8192)
    for got in launches(call, dict(call, capturing=True), few):
        assert all(n * threads < 2 ** 32 for _, grid, threads in got for n in grid)
    wide, narrow = launches(call, few)
    assert not is_compact(wide[0]) and wide[0][1] == (32768, 7, 64)
    assert is_compact(narrow[0]) and narrow[0][1] == (443 * 8192, 1, 1)


def test_row_blocks_of_many_heads_stay_within_the_launch(launches):
    """A launch holds at most 65535 row blocks x kv-heads: 960 rows of 14000 kv-heads fit it in four blocks of
    256, not in five of 192."""
    got, = launches(dict(ctx=[100], nodes=[240], hq=56000, hkv=14000, d=64))
    assert got[0][1:] == ((4 * 14000, 1, 1), 512)


def test_wide_trees_at_head_dim_64_keep_the_splits_of_two_workgroups_per_cu(launches):
    """The split length decides which maximum a row's probabilities are rounded against. Whatever the kernel,
    it is the shortest, in 64-token tiles, whose blocks of 256 rows stay within two a CU."""
    call = lambda batch, tokens, nodes, hkv=8: dict(ctx=[tokens - nodes] * batch, nodes=[nodes] * batch,
                                                    hq=4 * hkv, hkv=hkv, d=64)
    shapes = [(8, 8192, 64, 8), (8, 8192, 50, 8), (4, 8192, 100, 8), (1, 2048, 64, 8), (1, 2048, 100, 8),
              (16, 1024, 64, 4), (8, 4096, 48, 8), (2, 1024, 80, 8)]
    for (batch, tokens, nodes, hkv), got in zip(shapes, launches(*[call(*s) for s in shapes])):
        blocks = batch * hkv * -(-4 * nodes // 256)
        tiles = next(t for t in range(4, tokens // 64 + 1) if blocks * -(-tokens // (64 * t)) <= 512)
        (name, grid, threads), splits = got[0], -(-tokens // (64 * tiles))
        assert grid[1:] == (splits, batch), (batch, tokens, nodes)
        wide = -(-4 * nodes // -(-4 * nodes // 256)) > 192         # blocks of more than 192 rows, balanced
        small = batch * splits * hkv * -(-4 * nodes // 192) <= 256
        assert ("tree_attn_mfma" in name) == (wide and not small), (name, batch, tokens, nodes)


def test_fp32_launches_that_leave_the_last_round_idle_are_split(launches):
    """80 nodes on 8 kv-heads of four heads are ten 32-row blocks a kv-head: 640 blocks for eight
    sequences, of which 128 would fill a quarter of a second round of 512. They take splits; five
    sequences (400 blocks), sixteen (1280, 83 % of three rounds) and short ones do not."""
    call = lambda batch, tokens=1500, **kw: dict(dict(ctx=[tokens - 80] * batch, nodes=[80] * batch, hq=32, hkv=8,
                                                      d=128, dtype="f32"), **kw)
    eight, ragged, five, sixteen, short = [got[0] for got in launches(
        call(8), call(8, ctx=[1400, 400, 650, 100, 1300, 0, 1000, 300]), call(5), call(16), call(8, 1280))]
    assert eight[1] == (80, 4, 8)                   # 384-token splits
    assert is_compact(ragged) and ragged[1][0] > 640
    assert five[1] == (80, 1, 5)
    assert sixteen[1] == (80, 1, 16)
    assert short[1] == (80, 1, 8)


def test_ragged_launches_that_fit_are_not_listed(launches):
    """Where the CUs hold the full grid at one workgroup each there is nothing to gain from a list, nor at two
    each when the workgroups with work need that too."""
    call = lambda ctx, nodes, hkv, d: dict(ctx=ctx, nodes=[nodes] * len(ctx), hq=4 * hkv, hkv=hkv, d=d)
    one, half, two, more = [got[0] for got in launches(
        call([1708, 2854], 6, 8, 64),                      # 8 heads x 12 splits x 2
        call([2600, 900, 1000], 32, 8, 128),               # 8 x 11 x 3, of which 160 have work
        call([854, 1781, 1300, 1500], 100, 8, 64),         # two blocks of 8 heads x 8 x 4, 400
        call([854, 1781, 1300, 1500] * 2, 100, 8, 64))]    # twice as many
    assert not is_compact(one) and one[1] == (8, 12, 2)
    assert is_compact(half) and half[1] == (8 * (11 + 4 + 5), 1, 1)
    assert not is_compact(two) and two[1][0] * two[1][1] * two[1][2] <= 512
    assert is_compact(more)


@pytest.mark.parametrize("dtype,size", [("bf16", 2), ("f32", 4)])
def test_short_logits_rows_between_vector_boundaries_are_read_singly(launches, dtype, size):
    """Rows that all start at a 16-byte boundary take vectors whatever their length, others from 1280 entries."""
    vectors = lambda *rows: ["Lb1" in got[0][0].split("margins_kernel")[1][:10] for got in launches(
        *[dict(vocab=v, ld=ld, offset=off, dtype=dtype) for v, ld, off in rows])]
    assert vectors((1003, 1008, 0), (1003, 1003, 0), (1008, 1008, size), (1279, 1279, 0), (1281, 1281, 0),
                   (1280, 1280, size)) == [True, False, False, False, True, True]
