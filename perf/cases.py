"""The work that users of libcure have it do, as cases that can be timed and checked.

One decoding iteration of the verify-and-repair method is: the margin pass over
the draft block's logits and the repair tree built at its low-margin positions
("draft"), the target's attention over the tree's nodes, layer by layer
("attention"), the margin pass over the nodes' target logits with the
acceptance walk ("score"), and the commit of the winning path in every layer's
cache ("commit"). "verify" is the benchmark's step, one attention layer and then
the scoring, captured in a HIP graph once and replayed, as a latency-bound
decoding loop does with its fixed buffers. Each kind calls the package's own functions on tensors a serving
program holds at that point. Shapes are the package's configurations (a
Llama-3-8B-class target, chain 16, repair budgets of 0 to 64 nodes in branches
of depth 4) and the ranges its tests cover.
"""

import math
import random

import torch

import paper_2608_00531_amd as pc

CHAIN = 16
DEPTH = 4
MARGIN_SCALE = 1.0
_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _attention(name, dtype, batch, ctx_min, ctx_max, hq, hkv, d, chain, branches, depth):
    return dict(name=name, kind="attention", dtype=dtype, batch=batch, ctx_min=ctx_min,
                ctx_max=ctx_max, hq=hq, hkv=hkv, d=d, chain=chain, branches=branches, depth=depth)


def listed():
    return [
        # The smallest call there is: one short fp32 sequence, four heads, 12 nodes. All latency.
        _attention("attention_tiny_f32", "f32", 1, 128, 128, 4, 4, 64, 8, 2, 2),
        # One interactive user, 2k context, 32 nodes: the benchmark's default step.
        dict(_attention("verify_ctx2k_b1", "bf16", 1, 2048, 2048, 32, 8, 128, CHAIN, 4, DEPTH),
             kind="verify", vocab=128256),
        # A serving batch of sequences at different lengths, 48 nodes each.
        _attention("attention_ragged_b16", "bf16", 16, 1024, 4096, 32, 8, 128, CHAIN, 8, DEPTH),
        # Long documents: few sequences, 32k context, 32 nodes.
        _attention("attention_ctx32k_b4", "bf16", 4, 32768, 32768, 32, 8, 128, CHAIN, 4, DEPTH),
        # The widest tree of the budget sweep: 80 nodes at 8k context.
        _attention("attention_wide_b8", "bf16", 8, 8192, 8192, 32, 8, 128, CHAIN, 16, DEPTH),
        # A target with head dim 64 (smaller models), ragged batch, 48 nodes.
        _attention("attention_d64_b8", "bf16", 8, 1000, 4000, 32, 8, 64, CHAIN, 8, DEPTH),
        # Full-precision verification (reference runs, small fp32 targets), ragged batch.
        _attention("attention_f32_b4", "f32", 4, 500, 2000, 32, 8, 128, CHAIN, 4, DEPTH),
        # Scoring a serving batch: 768 node rows of target logits, with the acceptance walk.
        dict(name="score_ragged_b16", kind="score", dtype="bf16", batch=16, chain=CHAIN, branches=8,
             depth=DEPTH, vocab=128256),
        # A vocabulary that is no multiple of anything: every other row starts misaligned.
        dict(name="score_odd_vocab_b8", kind="score", dtype="bf16", batch=8, chain=CHAIN, branches=4,
             depth=DEPTH, vocab=50257),
        # The draft side of a batch: margins and gate over the block, then the repair tree.
        dict(name="draft_b8", kind="draft", dtype="bf16", batch=8, chain=CHAIN, branches=8,
             depth=DEPTH, vocab=128256),
        # The same with an fp32 draft head and a smaller vocabulary.
        dict(name="draft_f32_b4", kind="draft", dtype="f32", batch=4, chain=CHAIN, branches=4,
             depth=DEPTH, vocab=32000),
        # The end of an iteration: the walk, then the winning rows moved in all 32 layers.
        dict(name="commit_l32_b16", kind="commit", dtype="bf16", batch=16, ctx_min=200, ctx_max=500,
             hkv=8, d=128, layers=32, chain=CHAIN, branches=8, depth=DEPTH, vocab=128256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: 1 to 16 sequences, contexts of 100 to 32k tokens, chains of 4 to
    32 nodes with up to 16 branches of depth 1 to 4, vocabularies of 1000 to 152000 entries."""
    kind = rng.choice(["attention", "attention", "attention", "verify", "score", "score", "draft",
                       "commit"])
    chain = rng.randint(4, 32)
    depth = rng.randint(1, 4)
    branches = rng.randint(0, min(16, chain))
    batch = _log_int(rng, 1, 16)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    case = dict(kind=kind, dtype=dtype, batch=batch, chain=chain, branches=branches, depth=depth)
    if kind in ("attention", "verify"):
        hq, hkv = rng.choice([(32, 8), (32, 8), (32, 4), (16, 16), (8, 1), (12, 2)])
        d = rng.choice([64, 128])
        # At most what the largest listed case of the type reads and multiplies.
        nodes = chain + branches * depth
        tokens = (8000 if dtype == "f32" else 65536) * 8 // max(hkv, hq * nodes // 320)
        hi = max(100, min(32768, tokens // batch))
        a, b = sorted((_log_int(rng, 100, hi), _log_int(rng, 100, hi)))
        case.update(ctx_min=a, ctx_max=b, hq=hq, hkv=hkv, d=d)
    if kind in ("score", "verify", "draft"):
        rows = batch * (chain if kind == "draft" else chain + branches * depth)
        hi = min(152000, 90000000 // (rows * (2 if dtype == "f32" else 1)))
        case.update(vocab=_log_int(rng, 1000, hi))
    if kind == "draft":
        case.update(branches=max(1, branches))
    if kind == "commit":
        case.update(dtype="bf16", ctx_min=100, ctx_max=rng.randint(100, 500), hkv=rng.choice([1, 2, 4, 8]),
                    d=rng.choice([64, 128]), layers=rng.randint(1, 32), vocab=128256)
    return case


def _nodes(case):
    return case["chain"] + case["branches"] * case["depth"]


def _contexts(case):
    """The sequences' context lengths, spread over the case's range."""
    lo, hi = case["ctx_min"], case["ctx_max"]
    return [lo + int((hi - lo) * (((i + 1) * 0.6180339887498949) % 1.0)) for i in range(case["batch"])]


def _trees(case, rng):
    """Chains with branches at random positions: parents, tokens and the target's argmaxes, which
    follow the draft at 80 % of the nodes."""
    chain, depth, vocab = case["chain"], case["depth"], case.get("vocab", 128256)
    parents, tokens, targets, roots = [], [], [], []
    for _ in range(case["batch"]):
        parent = [i - 1 for i in range(chain)]
        for u in sorted(rng.sample(range(chain), case["branches"])):
            for t in range(depth):
                parent.append(u - 1 if t == 0 else len(parent) - 1)
        n = len(parent)
        token = [rng.randrange(vocab) for _ in range(n)]
        target = [rng.randrange(vocab) for _ in range(n + 1)]
        for i in reversed(range(n)):               # the lowest-numbered agreeing child wins
            if rng.random() < 0.8:
                target[parent[i] + 1] = token[i]
        parents.append(parent)
        tokens.append(token)
        roots.append(target[0])
        targets.append(target[1:])
    i32 = dict(dtype=torch.int32, device="cuda")
    return (torch.tensor(parents, **i32), torch.tensor(tokens, **i32), torch.tensor(targets, **i32),
            torch.tensor(roots, **i32))


def _logits(gen, shape, dtype, spike):
    """N(0, 3) with the entry `spike` of every row raised above the rest by 0.02 to 4."""
    x = torch.randn(shape, generator=gen, device="cuda", dtype=dtype).mul_(3.0)
    gap = torch.rand(shape[:2], generator=gen, device="cuda").mul_(3.98).add_(0.02)
    top = x.amax(dim=-1).float() + gap
    return x.scatter_(2, spike.long().unsqueeze(-1), top.to(dtype).unsqueeze(-1))


def prepare(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype, kind, batch, n = _DTYPES[case["dtype"]], case["kind"], case["batch"], _nodes(case)
    i32 = dict(dtype=torch.int32, device="cuda")
    state = dict(case=case, kind=kind, chain=case["chain"], depth=case["depth"],
                 budget=case["branches"] * case["depth"])
    if kind != "draft":
        parent, token, target, root = _trees(case, rng)
        state.update(parent=parent, token=token, target=target, root=root,
                     n_nodes=torch.full((batch,), n, **i32))
    if kind in ("attention", "verify", "commit"):
        ctx = _contexts(case)
        off, rows = [], 0
        for c in ctx:
            off.append(rows)
            rows += c + n
        state.update(ctx=ctx, kv_off=torch.tensor(off, dtype=torch.int64, device="cuda"),
                     ctx_len=torch.tensor(ctx, **i32))
        cache = (rows, case["hkv"], case["d"])
        if kind == "commit":
            cache = (case["layers"],) + cache
        state["k"] = torch.randn(cache, generator=gen, device="cuda", dtype=dtype)
        state["v"] = torch.randn(cache, generator=gen, device="cuda", dtype=dtype)
    if kind in ("attention", "verify"):
        state["q"] = torch.randn((batch, n, case["hq"], case["d"]), generator=gen, device="cuda", dtype=dtype)
        state["scale"] = 1.0 / math.sqrt(case["d"])
    if kind in ("score", "verify"):
        state["logits"] = _logits(gen, (batch, n, case["vocab"]), dtype, state["target"])
    if kind == "draft":
        chain = case["chain"]
        best = torch.randint(case["vocab"], (batch, chain), generator=gen, device="cuda")
        state["logits"] = _logits(gen, (batch, chain, case["vocab"]), dtype, best)
        state["chain_tok"] = best.to(torch.int32)
        state["suffix"] = None if case["depth"] == 1 else torch.randint(
            case["vocab"], (batch, chain, 5, case["depth"] - 1), generator=gen, **i32)
    if kind == "verify":
        _capture(state)
    return state


def _capture(s):
    """The step as a graph on a stream of its own, after one eager pass there."""
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        _attend(s), _score(s)
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            s["out"] = _attend(s), _score(s)
    torch.cuda.current_stream().wait_stream(stream)
    s["graph"] = graph


def _attend(s):
    ctx = s["ctx"]
    return pc.cure_tree_attn(s["q"], s["k"], s["v"], s["kv_off"], s["ctx_len"], s["n_nodes"],
                             s["parent"], ctx, [s["parent"].shape[1]] * len(ctx), s["scale"])


def _score(s):
    return pc.cure_margins_accept(s["logits"], s["parent"], s["token"], s["root"], s["n_nodes"],
                                  s["chain"], repair_budget=s["budget"], branch_depth=s["depth"])


def run(s):
    kind = s["kind"]
    if kind == "attention":
        return _attend(s)
    if kind == "verify":
        s["graph"].replay()
        return s["out"]
    if kind == "score":
        return _score(s)
    if kind == "draft":
        m = pc.cure_margins(s["logits"], s["chain"], repair_budget=s["budget"], branch_depth=s["depth"])
        # Every position may get a branch, so the budget is always spent and every node written.
        tree = pc.cure_repair_tree(s["logits"], m["margin"], m["ufp_pos"], m["ufp_cnt"], s["chain_tok"],
                                   s["budget"], s["depth"], MARGIN_SCALE, suffix=s["suffix"])
        return m, tree
    a = pc.cure_accept(s["parent"], s["token"], s["target"], s["root"], s["n_nodes"], s["chain"])
    c = pc.cure_commit(s["k"], s["v"], s["kv_off"], s["ctx_len"], s["n_nodes"], a["path"],
                       a["acc_len"], s["token"], a["bonus"], s["chain"])
    return a, c, s["k"], s["v"]


def work(case):
    eb = 4 if case["dtype"] == "f32" else 2
    kind, batch, n = case["kind"], case["batch"], _nodes(case)
    nbytes = flops = 0
    if kind in ("attention", "verify"):
        tokens = sum(c + n for c in _contexts(case))
        hq, d = case["hq"], case["d"]
        # K and V once; q and o; the log-sum-exps; the tree.
        nbytes += tokens * case["hkv"] * d * 2 * eb + batch * n * hq * (2 * d * eb + 4) + batch * n * 4
        # Two multiply-adds per head dim, node and visible row (a root path is about half a chain).
        flops += 4 * d * hq * n * sum(c + case["chain"] // 2 for c in _contexts(case))
    if kind in ("score", "verify", "draft"):
        rows = batch * (case["chain"] if kind == "draft" else n)
        nbytes += rows * (case["vocab"] * eb + 24) + (0 if kind == "draft" else batch * n * 12)
        flops += 4 * rows * case["vocab"]          # two comparisons, an exponential and a sum
    if kind == "draft":
        nbytes += batch * case["vocab"] * eb + batch * n * 12     # at least one row ranked
    if kind == "commit":
        # About three of five accepted rows sit in place already; two rows read and written.
        nbytes += batch * (2 * 2 * 2 * case["layers"] * case["hkv"] * case["d"] * eb + n * 24)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "commit":
        return "exact"                             # rows moved and whole numbers
    if case["kind"] in ("attention", "verify") and case["dtype"] == "bf16":
        return {"rel": 1e-2}                       # bf16 probabilities and outputs
    return {"rel": 1e-5}                           # fp32 sums; indices and walks are whole numbers


def _exact_attention(s):
    case = s["case"]
    n, hq, hkv, d = _nodes(case), case["hq"], case["hkv"], case["d"]
    g = hq // hkv
    f64 = dict(dtype=torch.float64, device="cuda")
    out = torch.empty(case["batch"], n, hq, d, **f64)
    lse = torch.empty(case["batch"], n, hq, **f64)
    parents = s["parent"].tolist()
    for b, c in enumerate(s["ctx"]):
        seen = [[False] * n for _ in range(n)]
        for i, p in enumerate(parents[b]):
            if p >= 0:
                seen[i] = list(seen[p])
            seen[i][i] = True
        hidden = ~torch.tensor(seen, device="cuda").repeat_interleave(g, dim=0)
        at = int(s["kv_off"][b])
        for h in range(hkv):
            q = s["q"][b, :, h * g:(h + 1) * g].double().reshape(n * g, d)
            k = s["k"][at:at + c + n, h].double()
            x = (q @ k.t().contiguous()) * s["scale"]
            x[:, c:].masked_fill_(hidden, -math.inf)
            o = torch.softmax(x, dim=-1) @ s["v"][at:at + c + n, h].double()
            out[b, :, h * g:(h + 1) * g] = o.reshape(n, g, d)
            lse[b, :, h * g:(h + 1) * g] = torch.logsumexp(x, dim=-1).reshape(n, g)
    return out, lse, None


def _exact_margins(logits):
    rows = [x.double() for x in logits]
    top = torch.stack([x.topk(2, dim=-1).values for x in rows])
    return {"top1_val": top[..., 0], "top2_val": top[..., 1], "margin": top[..., 0] - top[..., 1],
            "lse": torch.stack([torch.logsumexp(x, dim=-1) for x in rows])}


def exact(case, seed):
    kind = case["kind"]
    if kind == "commit":
        return None                                # nothing is computed: rows move
    s = prepare(case, seed)
    if kind == "attention":
        return _exact_attention(s)
    if kind == "verify":
        return _exact_attention(s), _exact_margins(s["logits"])
    if kind == "score":
        return _exact_margins(s["logits"])
    return _exact_margins(s["logits"]), {}
