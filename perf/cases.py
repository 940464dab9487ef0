"""The work that programs have this library do, as cases that can be timed and compared.

A case names a model (its operations), the shape of its graphs, sizes, a data type and a task:

  infer     a new batch arrives: schedule it and run the forward pass (a server's request)
  batch     a new batch arrives: schedule it, forward, backward (one step of dynamic batching in training)
  graph     the same schedule again: forward and backward as one recorded step
  train     a whole training step: loss head on every node, backward, Adam, weights packed again
  schedule  the schedule alone
  typed     the paper-form schedule alone (typed states, pass-throughs)

`prepare` makes the inputs from the seed, `run` is one pass, `exact` is the same pass in 64 bits in plain torch.
"""
import ctypes
import math
import zlib

import numpy as np
import torch

from paper_1702_02181_amd import fold as F
from paper_1702_02181_amd import gen, runner

GATES = {"embed": 0, "treernn": 1, "treelstm": 5, "lstm": 4, "proj": 1, "score": 0, "sum": 0, "out": 0}
KIND = {"embed": F.FOLD_EMBED, "treernn": F.FOLD_TREERNN, "treelstm": F.FOLD_TREELSTM, "lstm": F.FOLD_LSTM,
        "proj": F.FOLD_PROJ, "score": F.FOLD_ATTN_SCORE, "sum": F.FOLD_ATTN_SUM, "out": F.FOLD_ATTN_OUT}

# model -> [(kind, arity, reads a leaf-table row, parameter set)] and [(kind, reads the table, children)] of the sets
MODELS = {
    "treernn": ([("embed", 0, 1, 0), ("treernn", 2, 0, 1)], [("embed", 1, 0), ("treernn", 0, 2)]),
    "treelstm": ([("treelstm", 0, 1, 0), ("treelstm", 2, 0, 0)], [("treelstm", 1, 2)]),
    "mixed": ([("lstm", 1, 1, 0), ("treelstm", 2, 0, 1), ("proj", 1, 0, 2)],
              [("lstm", 1, 1), ("treelstm", 0, 2), ("proj", 0, 1)]),
    "attention": ([("embed", 0, 1, 0), ("proj", 1, 0, 1), ("score", 1, 0, 2), ("sum", 2, 0, 3), ("out", 1, 0, 4),
                   ("proj", 1, 0, 5)],
                  [("embed", 1, 0), ("proj", 0, 1), ("score", 0, 1), ("sum", 0, 2), ("out", 0, 1), ("proj", 0, 1)]),
}


def _case(name, task, model, shape, dtype, hidden, in_dim, graphs, lo, hi, vocab=0, **more):
    """vocab 0: a table row of its own for every leaf; lo..hi: leaves (items, chain steps) of a graph."""
    c = dict(task=task, model=model, shape=shape, dtype=dtype, hidden=hidden, in_dim=in_dim, graphs=graphs, lo=lo,
             hi=hi, vocab=vocab, dropout=0.0, classes=0, noalloc=False)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A small model's request: eight short sentences through a TreeRNN, where launches and latency count.
        _case("serve_rnn_b8_h64_f32", "infer", "treernn", "random", "f32", 64, 64, 8, 2, 16, 100),
        # The paper's timing benchmark (Table 1, full dynamic) at batch size 1: one tree of 64 leaves.
        _case("serve_tree_b1_h1024_f32", "infer", "treelstm", "random", "f32", 1024, 1024, 1, 64, 64, 10000),
        # The same at batch size 256: a loaded server, every tree with a shape of its own.
        _case("serve_tree_b256_h1024_f32", "infer", "treelstm", "random", "f32", 1024, 1024, 256, 64, 64, 10000),
        # Sentiment trees served in bf16 by a program that may not allocate workspaces.
        _case("serve_sentiment_b32_h300_bf16", "infer", "treelstm", "random", "bf16", 300, 300, 32, 5, 60, 20000,
              noalloc=True),
        # Fixed shape, recorded step: 256 complete trees of 256 leaves, fp32, each leaf with its own input row.
        _case("step_balanced_h256_f32", "graph", "treelstm", "balanced", "f32", 256, 256, 256, 256, 256),
        # Sentiment trees in training with recurrent dropout: a new batch scheduled, forward, backward.
        _case("batch_sentiment_h300_bf16", "batch", "treelstm", "random", "bf16", 300, 300, 1024, 5, 60, 20000,
              dropout=0.25),
        # The whole training step on such trees: a class on every node, Adam on all weights and the table.
        _case("train_sentiment_h300_bf16", "train", "treelstm", "random", "bf16", 300, 300, 1024, 5, 60, 20000,
              classes=5),
        # Mixed operations: LSTM chains under a reduce tree with projections; many narrow levels.
        _case("batch_mixed_h512_bf16", "batch", "mixed", "reduce", "bf16", 512, 128, 512, 1, 100),
        # The largest: two million nodes, balanced trees and caterpillars with shared sub-expressions.
        _case("step_dag_h1024_bf16", "graph", "treelstm", "dag", "bf16", 1024, 1024, 4096, 200, 511, 20000),
        # Feed-forward attention over sequences: memory-bound operations and one projection per item.
        _case("step_attention_h256_bf16", "graph", "attention", "items", "bf16", 256, 256, 1024, 50, 100),
        # Scheduling by itself, for the largest batch: index work over two million nodes, 512 levels.
        _case("schedule_dag_2m", "schedule", "treelstm", "dag", "bf16", 64, 64, 4096, 200, 511, 20000),
        # The paper-form schedule of a batch of sentiment trees (word ids, embeddings, h and c as typed states).
        _case("typed_sentiment_b1024", "typed", "treelstm", "random", "bf16", 64, 64, 1024, 5, 60, 20000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    task = rng.choice(["infer", "infer", "batch", "batch", "graph", "train", "schedule", "typed"])
    dtype = rng.choice(["f32", "bf16"])
    model = {"infer": rng.choice(["treernn", "treelstm", "mixed"]), "batch": rng.choice(["treelstm", "mixed", "attention"]),
             "graph": rng.choice(["treelstm", "mixed", "attention"]), "train": "treelstm", "schedule": "treelstm",
             "typed": "treelstm"}[task]
    hidden = _log_int(rng, 48, 1024)
    if rng.random() < 0.5:  # widths are often multiples of 64
        hidden = max(64, hidden // 64 * 64)
    if model == "attention":
        hidden = min(hidden, 512)
    most = {"infer": 1024, "batch": 2048, "graph": 2048, "train": 1024, "schedule": 4096, "typed": 2048}[task]
    graphs = _log_int(rng, 1, most)
    if model == "mixed":
        shape, lo, hi, vocab = "reduce", 1, rng.randint(10, 100), 0
    elif model == "attention":
        shape, lo, hi, vocab = "items", rng.randint(1, 50), rng.randint(51, 100), 0
    else:
        shape = rng.choice(["random", "random", "balanced", "dag"] if task in ("batch", "graph", "schedule") else
                           ["random", "random", "balanced"])
        lo = rng.randint(2, 60)
        hi = lo if shape == "balanced" else rng.randint(lo, 130 if shape == "random" else 300)
        vocab = _log_int(rng, 100, 20000)
        vocab = vocab if task == "train" else rng.choice([0, vocab])
    in_dim = hidden if model in ("treernn", "attention") else rng.choice([hidden, _log_int(rng, 50, 512)])
    while graphs > 1 and graphs * hi * (hidden + 64) ** 2 > 1.0e11:  # no more than the listed cases cost
        graphs = (graphs + 1) // 2
    dropout = rng.choice([0.0, 0.25]) if task == "batch" and model in ("treelstm", "mixed") else 0.0
    return _case(None, task, model, shape, dtype, hidden, in_dim, graphs, lo, hi, vocab, dropout=dropout,
                 classes=rng.choice([2, 5, 10]) if task == "train" and hidden <= 800 else 5,
                 noalloc=task == "infer" and rng.random() < 0.3)


# ---- graphs ---------------------------------------------------------------------------------------------------

def _reduce(rng, leaves, how):
    """Binary trees over leaves[g] items each, the internal nodes of every tree numbered in post-order.

    how[g]: 0 the left subtree gets U{1..n-1} items, 1 floor(n/2), 2 all but one.  Returns left, right and last of
    every internal node: a child is the item's number, or ~ the internal node's; last is the node's last item."""
    leaves = np.asarray(leaves, np.int64)
    how = np.broadcast_to(np.asarray(how, np.int64), leaves.shape)
    total = int((leaves - 1).sum())
    left, right, last = (np.zeros(total, np.int64) for _ in range(3))
    a = np.cumsum(leaves) - leaves
    base = np.cumsum(leaves - 1) - (leaves - 1)
    keep = leaves > 1
    a, n, base, how = a[keep], leaves[keep], base[keep], how[keep]
    while a.size:
        k = np.where(how == 0, 1 + (rng.random(n.size) * (n - 1)).astype(np.int64), np.where(how == 1, n // 2, n - 1))
        k = np.clip(k, 1, n - 1)
        root = base + n - 2
        left[root] = np.where(k == 1, a, ~(base + k - 2))
        right[root] = np.where(n - k == 1, a + k, ~(base + n - 3))
        last[root] = a + n - 1
        l, r = k > 1, n - k > 1
        a, n, base, how = (np.concatenate(x) for x in ((a[l], (a + k)[r]), (k[l], (n - k)[r]), (base[l], (base + k - 1)[r]),
                                                       (how[l], how[r])))
    return left, right, last


def _tree(rng, leaves, how, rows, share=0.0):
    """Trees whose items are leaf nodes (operation 0), all in post-order; share: the part of the leaf slots that name
    an earlier node of their graph instead (their leaves are gone), which makes shared sub-expressions."""
    leaves = np.asarray(leaves, np.int64)
    left, right, last = _reduce(rng, leaves, how)
    count = int(leaves.sum())
    before = np.concatenate([[0], np.cumsum(np.bincount(last, minlength=count))])[:count]
    leaf_at = np.arange(count) + before
    node_at = last + 1 + np.arange(last.size)
    at = lambda x: np.where(x >= 0, leaf_at[np.maximum(x, 0)], node_at[np.maximum(~x, 0)] if node_at.size else 0)  # noqa: E731
    n = count + last.size
    op = np.zeros(n, np.int64)
    op[node_at] = 1
    inp = np.full(n, -1, np.int64)
    inp[leaf_at] = rows
    kids = np.stack([at(left), at(right)], 1) if last.size else np.zeros((0, 2), np.int64)
    sizes = 2 * leaves - 1
    if share > 0 and kids.size:
        start = np.repeat(np.cumsum(sizes) - sizes, leaves - 1)
        slot = (op[kids] == 0) & (rng.random(kids.shape) < share)
        row, side = np.nonzero(slot)
        gone = np.zeros(n, bool)
        gone[kids[row, side]] = True
        source = np.nonzero((rng.random(n) < 0.15) & ~gone)[0]  # the nodes that are shared
        hi = np.searchsorted(source, node_at[row])
        lo = np.maximum(np.searchsorted(source, start[row]), hi - 16)
        ok = hi > lo
        gone[kids[row, side][~ok]] = False
        pick = hi - 1 - (rng.random(row.size) * np.maximum(hi - lo, 1)).astype(np.int64)
        kids[row[ok], side[ok]] = source[pick[ok]]
        new = np.cumsum(~gone) - 1
        op, inp, kids = op[~gone], inp[~gone], new[kids]
        cut = np.concatenate([[0], np.cumsum(sizes)])
        sizes = np.diff(np.concatenate([[0], np.cumsum(~gone)])[cut])
    counts = np.where(op == 1, 2, 0)
    return sizes, op, counts, kids.reshape(-1), inp


def _mixed(rng, steps, rows, proj):
    """An LSTM chain over `steps` rows, a halving reduce over its states, a projection above a part of its nodes."""
    steps = np.asarray(steps, np.int64)
    left, right, _ = _reduce(rng, steps, 1)
    internal = steps - 1
    tree = np.repeat(np.arange(steps.size), internal)
    has = rng.random(tree.size) < proj
    upto = np.cumsum(1 + has)  # internal nodes and projections, up to and with each node's own
    made = np.concatenate([[0], upto])
    ends = np.cumsum(internal)
    sizes = steps + made[ends] - made[ends - internal]
    start = np.cumsum(sizes) - sizes
    item = np.arange(int(steps.sum()))
    of = np.repeat(np.arange(steps.size), steps)
    step = item - np.repeat(np.cumsum(steps) - steps, steps)
    chain_at = start[of] + step
    shift = (start + steps)[tree] - made[(ends - internal)[tree]]
    node_at = shift + made[:-1]
    value_at = node_at + has
    at = lambda x: np.where(x >= 0, chain_at[np.maximum(x, 0)], value_at[np.maximum(~x, 0)])  # noqa: E731
    n = int(sizes.sum())
    op, inp = np.zeros(n, np.int64), np.full(n, -1, np.int64)
    one, two = np.full(n, -1, np.int64), np.full(n, -1, np.int64)
    inp[chain_at] = rows
    one[chain_at] = np.where(step > 0, chain_at - 1, -1)
    counts = np.ones(n, np.int64)
    if tree.size:
        op[node_at], counts[node_at] = 1, 2
        one[node_at], two[node_at] = at(left), at(right)
        op[value_at[has]], one[value_at[has]] = 2, node_at[has]
    both = np.stack([one, two], 1)
    return sizes, op, counts, both[np.arange(2)[None, :] < counts[:, None]], inp


def _items(rng, items, rows):
    """Attention: every item an embedding, a projection and a score; a halving merge, the output, a projection."""
    items = np.asarray(items, np.int64)
    left, right, _ = _reduce(rng, items, 1)
    sizes = 4 * items + 1
    start = np.cumsum(sizes) - sizes
    of = np.repeat(np.arange(items.size), items)
    i = np.arange(int(items.sum())) - np.repeat(np.cumsum(items) - items, items)
    embed = start[of] + 3 * i
    tree = np.repeat(np.arange(items.size), items - 1)
    rank = np.arange(tree.size) - np.repeat(np.cumsum(items - 1) - (items - 1), items - 1)
    sum_at = (start + 3 * items)[tree] + rank
    at = lambda x: np.where(x >= 0, embed[np.maximum(x, 0)] + 2, sum_at[np.maximum(~x, 0)] if sum_at.size else 0)  # noqa: E731
    n = int(sizes.sum())
    op, inp, counts = np.zeros(n, np.int64), np.full(n, -1, np.int64), np.ones(n, np.int64)
    one, two = np.full(n, -1, np.int64), np.full(n, -1, np.int64)
    inp[embed], counts[embed] = rows, 0
    op[embed + 1], one[embed + 1] = 1, embed
    op[embed + 2], one[embed + 2] = 2, embed + 1
    if tree.size:
        op[sum_at], counts[sum_at] = 3, 2
        one[sum_at], two[sum_at] = at(left), at(right)
    out = start + sizes - 2
    op[out], one[out] = 4, out - 1
    op[out + 1], one[out + 1] = 5, out
    both = np.stack([one, two], 1)
    return sizes, op, counts, both[np.arange(2)[None, :] < counts[:, None]], inp


def _typed(sizes, op, counts, kids):
    """A Tree-LSTM batch as typed graphs: word id (type 0) -> embed -> leaf cell; internal cells read h and c (type 1)
    of both children."""
    width = np.where(op == 0, 3, 1)
    ends = np.cumsum(width)
    value = ends - 1
    n = int(ends[-1])
    node_op = np.full(n, 2, np.int64)
    inputs = np.full(n, 4, np.int64)
    leaf = value[op == 0]
    node_op[leaf], node_op[leaf - 1], node_op[leaf - 2] = 1, 0, -1
    inputs[leaf], inputs[leaf - 1], inputs[leaf - 2] = 1, 1, 0
    ptr = np.concatenate([[0], np.cumsum(inputs)])
    node, slot = np.zeros(int(ptr[-1]), np.int64), np.zeros(int(ptr[-1]), np.int64)
    node[ptr[leaf]], node[ptr[leaf - 1]] = leaf - 1, leaf - 2
    inner = ptr[value[op == 1]]
    pair = value[kids].reshape(-1, 2)
    for k in range(4):
        node[inner + k], slot[inner + k] = pair[:, k // 2], k % 2
    graph_ptr = np.concatenate([[0], ends])[np.concatenate([[0], np.cumsum(sizes)])]
    return graph_ptr, node_op, ptr, node, slot


# ---- inputs ---------------------------------------------------------------------------------------------------

def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _ld(width):
    return (width + 63) // 64 * 64  # the rows of pools and tables (fold_row_ld)


def _padded(x):
    out = torch.zeros((x.shape[0], _ld(x.shape[1])), dtype=x.dtype, device=x.device)
    out[:, :x.shape[1]] = x
    return out


def _batch(case, seed):
    """The graphs of a case, as numpy arrays: the case decides how many of which shapes there are (so that arrays keep
    their sizes), the seed in which order they come, which child is the left one, and the rows that the leaves read."""
    fixed = np.random.default_rng(zlib.crc32(repr(sorted((k, v) for k, v in case.items() if k != "name")).encode()))
    rng = np.random.default_rng(seed)
    b, lo, hi = case["graphs"], case["lo"], case["hi"]
    sizes = fixed.integers(lo, hi + 1, b)
    how = {"random": 0, "balanced": 1, "dag": 1}.get(case["shape"], 1)
    if case["shape"] == "dag":  # balanced trees of 256 leaves (fewer in a small case) and caterpillars, in turn
        sizes = np.where(np.arange(b) % 2 == 0, min(256, hi), sizes + 1)
        how = np.where(np.arange(b) % 2 == 0, 1, 2)
    items = int(sizes.sum())
    if case["model"] == "mixed":
        sizes, op, counts, kids, reads = _mixed(fixed, sizes, 1, 0.2)
    elif case["model"] == "attention":
        sizes, op, counts, kids, reads = _items(fixed, sizes, 1)
    else:
        sizes, op, counts, kids, reads = _tree(fixed, sizes, how, 1, 0.4 if case["shape"] == "dag" else 0.0)
    order = rng.permutation(sizes.size)
    start, ptr = np.cumsum(sizes) - sizes, np.cumsum(counts) - counts
    node = _ranges(start[order], sizes[order])
    new = np.empty(node.size, np.int64)
    new[node] = np.arange(node.size)
    kids = np.where(kids >= 0, new[np.maximum(kids, 0)], -1)[_ranges(ptr[node], counts[node])]
    sizes, op, counts, reads = sizes[order], op[node], counts[node], reads[node] >= 0
    pair = (np.cumsum(counts) - counts)[counts == 2]
    pair = pair[rng.random(pair.size) < 0.5]
    kids[pair], kids[pair + 1] = kids[pair + 1], kids[pair]
    inp = np.full(node.size, -1, np.int64)
    leaves = int(reads.sum())
    if case["vocab"]:  # word frequencies follow Zipf's law
        p = np.cumsum(1.0 / np.arange(1, case["vocab"] + 1))
        inp[reads] = np.minimum(np.searchsorted(p, rng.random(leaves) * p[-1]), case["vocab"] - 1)
    else:
        inp[reads] = np.arange(leaves)
    return (sizes, op, counts, kids, inp), case["vocab"] or items


def _ranges(start, count):
    """start[i] .. start[i] + count[i] - 1, one after the other."""
    return np.repeat(start - (np.cumsum(count) - count), count) + np.arange(int(count.sum()))


def _inputs(case, seed, values=True):
    (sizes, op, counts, kids, inp), table_rows = _batch(case, seed)
    gpu = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.int32)).cuda()  # noqa: E731
    d = {"N": op.size, "rows": table_rows, "roots": int(case["graphs"])}
    d["ops"] = MODELS[case["model"]][0]
    if case["task"] == "typed":
        d["csr"] = [gpu(x) for x in _typed(sizes, op, counts, kids)]
        return d
    d["csr"] = [gpu(np.concatenate([[0], np.cumsum(sizes)])), gpu(op), gpu(np.concatenate([[0], np.cumsum(counts)])),
                gpu(kids), gpu(inp)]
    if not values or case["task"] == "schedule":
        return d
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    dt, H = _dtype(case), case["hidden"]
    uniform = lambda *s: torch.rand(s, generator=g, device="cuda") * 0.2 - 0.1  # noqa: E731
    normal = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    d["sets"] = []
    for kind, reads, arity in MODELS[case["model"]][1]:
        width = GATES[kind] * H if GATES[kind] else 1
        d["sets"].append({
            "kind": KIND[kind], "in_dim": case["in_dim"] if reads else 0, "arity": arity,
            "W_in": uniform(case["in_dim"], width).to(dt) if reads and kind != "embed" else None,
            "W_rec": uniform(arity * H, width).to(dt) if arity and kind not in ("sum", "out") else None,
            "bias": uniform(width) if kind not in ("embed", "sum", "out") else None})
    d["table"] = _padded((normal(table_rows, case["in_dim"]) * (0.1 if case["vocab"] else 1.0)).to(dt))
    if case["task"] != "infer":
        d["dh_roots"] = _padded(normal(d["roots"], H))
    if case["dropout"]:
        keep = torch.rand((d["N"], H), generator=g, device="cuda") >= case["dropout"]
        d["mask"] = _padded(keep.float() / (1.0 - case["dropout"]))
    if case["task"] == "train":
        d["labels"] = torch.randint(0, case["classes"], (d["N"],), generator=g, device="cuda", dtype=torch.int32)
        d["W_cls"], d["b_cls"] = 0.1 * normal(H, case["classes"]), torch.zeros(case["classes"], device="cuda")
    return d


class _View:
    """A device array that a schedule owns, as a tensor without a copy; it keeps the schedule alive."""

    def __init__(self, owner, at, count):
        at = at if isinstance(at, int) else ctypes.cast(at, ctypes.c_void_p).value
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (count,), "typestr": "<i4", "data": (at or 0, False), "version": 2}


def _view(owner, at, count):
    if not count:
        return torch.zeros(0, dtype=torch.int32, device="cuda")
    t = torch.as_tensor(_View(owner, at, count), device="cuda")
    t.owner = owner
    return t


def _op_table(case):
    return [(KIND[k], a, i, s) for k, a, i, s in MODELS[case["model"]][0]]


def prepare(case, seed):
    d = _inputs(case, seed)
    s = {"task": case["task"], "csr": d["csr"], "rows": d["rows"], "ops": _op_table(case)}
    if case["task"] == "schedule":
        return s
    if case["task"] == "typed":
        s["ops"] = [([0], [1]), ([1], [1, 1]), ([1, 1, 1, 1], [1, 1])]
        return s
    if case["task"] == "train":
        return dict(s, step=_train_step(case, d))
    dt, H = _dtype(case), case["hidden"]
    ld = F.fold_row_ld(H)
    s["packed"] = F.Packed(F.FOLD_BF16 if dt == torch.bfloat16 else F.FOLD_F32, H, d["sets"])
    s["table"], s["mask"], s["dh_roots"], s["noalloc"] = d["table"], d.get("mask"), d.get("dh_roots"), case["noalloc"]
    s["h"] = torch.zeros((d["N"], ld), dtype=dt, device="cuda")
    s["c"] = torch.zeros((d["N"], ld), device="cuda")
    s["out"] = torch.zeros((d["roots"], ld), dtype=dt, device="cuda")
    sched = F.Schedule(*s["csr"], s["ops"], s["rows"])
    fwd, bwd = F.fold_workspace_size(sched.handle, s["packed"].handle)
    s["ws"] = torch.empty(max(1, (0 if case["noalloc"] else fwd) if case["task"] == "infer" else bwd), dtype=torch.uint8,
                          device="cuda")
    if case["task"] == "infer":
        return s
    # all gradients in one buffer, each on a 256-byte boundary; the table's too where the table is a vocabulary's
    shapes = []
    for p in d["sets"]:
        shapes += [p["W_in"], p["W_rec"], p["bias"]]
    shapes.append(s["table"] if case["vocab"] else None)
    joint = KIND["score"]  # the scorer's bias gradient is zero up to rounding: it is compared with its vector's
    sizes = [0 if t is None else (t.numel() + 63) // 64 * 64 for t in shapes]
    s["flat"] = torch.zeros(max(1, sum(sizes)), device="cuda")
    views, at, s["grads"] = [], 0, {}
    for k, (t, n) in enumerate(zip(shapes, sizes)):
        views.append(None if t is None else s["flat"][at:at + t.numel()].view(t.shape))
        if t is not None and not (k // 3 < len(d["sets"]) and d["sets"][k // 3]["kind"] == joint):
            s["grads"]["d%d" % k] = views[-1]
        elif t is not None and k % 3 == 1:
            s["grads"]["d%d" % k] = s["flat"][at:at + n + 1]
        at += n
    s["c_grads"] = F.make_grads([tuple(views[3 * k:3 * k + 3]) for k in range(len(d["sets"]))], views[-1])
    if case["task"] == "graph":
        s["sched"] = sched
        s["graph"] = F.StepGraph(sched, s["packed"], s["table"], s["rows"], s["h"], s["c"], s["out"], s["ws"], bwd,
                                 backward=True, dh_roots=s["dh_roots"], grads=s["c_grads"], zero_grads=True)
    return s


def _train_step(case, d):
    host = lambda x, dt=np.float32: x.float().cpu().numpy().astype(dt)  # noqa: E731
    ints = [x.cpu().numpy() for x in d["csr"]]
    params = [gen.ParamSet(p["kind"], p["in_dim"], p["arity"], None if p["W_in"] is None else host(p["W_in"]),
                           None if p["W_rec"] is None else host(p["W_rec"]),
                           np.zeros(0, np.float32) if p["bias"] is None else host(p["bias"])) for p in d["sets"]]
    w = gen.Workload("train", case["dtype"], case["hidden"], *ints, [gen.OpSpec(*o) for o in _op_table(case)], params,
                     host(d["table"])[:, :case["in_dim"]], host(d["dh_roots"])[:, :case["hidden"]])
    step = runner.TrainStep(w, d["labels"].cpu().numpy(), case["classes"], True)
    step.W_cls.copy_(d["W_cls"])
    step.b_cls.copy_(d["b_cls"])
    return step


# ---- one pass -------------------------------------------------------------------------------------------------

def run(state):
    s, task = state, state["task"]
    if task == "graph":
        s["graph"].launch()
    elif task == "train":
        t = s["step"]
        t.step()
        return {"loss": t.node_loss, "h": t.dev.h_pool, "weights": [x[0] for x in t.tensors],
                "grads": [x[2] for x in t.tensors]}
    elif task == "typed":
        sched = F.TypedSchedule(*s["csr"], s["ops"], 2)
        i, n = sched.info, sched.num_nodes
        nb = i.num_batches
        return {k: _view(sched, getattr(i, k), c) for k, c in (
            ("depth", n), ("batch_depth", nb), ("batch_op", nb), ("batch_rows", nb), ("batch_gather_off", nb),
            ("batch_item_begin", nb), ("item_node", i.num_items), ("gather", i.num_gather),
            ("pass_node", i.num_passes), ("pass_slot", i.num_passes), ("pass_depth", i.num_passes),
            ("state_size", (i.num_levels + 1) * i.num_types), ("edge_index", sched.num_edges))}
    else:
        s["sched"] = sched = F.Schedule(*s["csr"], s["ops"], s["rows"])
        if task == "schedule":
            i = sched.info
            n, e, ng = i.num_nodes, i.num_edges, i.num_groups
            return {k: _view(sched, getattr(i, k), c) for k, c in (
                ("depth", n), ("node_pos", n), ("pos_node", n), ("level_ptr", i.num_levels + 1), ("group_level", ng),
                ("group_op", ng), ("group_row_begin", ng), ("group_rows", ng), ("group_idx_off", ng),
                ("child_pos", e), ("input_idx", n), ("root_pos", i.num_roots))}
        if s["noalloc"]:
            F.fold_forward_noalloc(sched.handle, s["packed"].handle, s["table"], s["rows"], s["h"], s["c"], s["out"])
            return {"roots": s["out"], "h": s["h"], "c": s["c"]}
        fwd, bwd = F.fold_workspace_size(sched.handle, s["packed"].handle)
        need = fwd if task == "infer" else bwd
        if need > s["ws"].numel():
            s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        args = (sched.handle, s["packed"].handle, s["table"], s["rows"], s["h"], s["c"])
        if task == "infer":
            F.fold_forward(*args, s["out"], s["ws"], need)
            return {"roots": s["out"], "h": s["h"], "c": s["c"]}
        s["flat"].zero_()
        if s["mask"] is None:
            F.fold_forward(*args, s["out"], s["ws"], need)
            F.fold_backward(*args, s["dh_roots"], None, s["c_grads"], None, None, s["ws"], need)
        else:
            F.fold_forward_dropout(*args, s["out"], s["mask"], s["ws"], need)
            F.fold_backward_dropout(*args, s["mask"], s["dh_roots"], None, s["c_grads"], None, None, s["ws"], need)
    return {"roots": s["out"], "h": s["h"], "c": s["c"], **s["grads"]}


# ---- what a pass needs, and how close its results are ---------------------------------------------------------

def work(case):
    """Expected over the graphs that `prepare` draws: CSR, weights and rows read once, states and gradients written
    once; the products of the cells (a Tree-LSTM leaf has three gates that count)."""
    b, H, D, H_b = case["graphs"], case["hidden"], case["in_dim"], 2 if case["dtype"] == "bf16" else 4
    mean = (case["lo"] + case["hi"]) / 2.0
    if case["shape"] == "dag":
        mean = (min(256, case["hi"]) + mean + 1) / 2.0
    leaves, inner = b * mean, b * (mean - 1)
    if case["model"] == "treelstm":
        live = leaves * (0.6 if case["shape"] == "dag" else 1.0)
        nodes, edges = live + inner, 2 * inner
        rec, leaf, weights = 2.0 * inner * 2 * H * 5 * H, 2.0 * live * D * 3 * H, (D + 2 * H) * 5 * H
    elif case["model"] == "treernn":
        nodes, edges, leaf = leaves + inner, 2 * inner, 0.0
        rec, weights = 2.0 * inner * 2 * H * H, 2 * H * H
    elif case["model"] == "mixed":
        nodes, edges = leaves + 1.2 * inner, leaves + 2.2 * inner
        rec = 2.0 * leaves * H * 4 * H + 2.0 * inner * 2 * H * 5 * H + 0.4 * inner * H * H
        leaf, weights = 2.0 * leaves * D * 4 * H, (D + H) * 4 * H + 10 * H * H + H * H
    else:
        nodes, edges, leaf = 3 * leaves + inner + 2 * b, 2 * leaves + 2 * inner + 2 * b, 0.0
        rec, weights = 2.0 * (leaves + b) * H * H + 8.0 * leaves * H, 2 * H * H + H
    csr = 4.0 * (b + 4 * nodes + edges)
    if case["task"] == "schedule":  # the arrays of fold_sched_info
        return {"bytes": csr + 4.0 * (4 * nodes + edges + b), "flops": 0}
    if case["task"] == "typed":  # three nodes a leaf; gather and edge index, the nodes' depths and the batches' items
        nodes, edges = 3 * leaves + inner, 2 * leaves + 4 * inner
        return {"bytes": 4.0 * (2 * nodes + 2 * edges + 2 * nodes + 2 * edges), "flops": 0}
    table = min(case["vocab"] or leaves, leaves) * D
    states = nodes * H * (H_b + 4.0) + b * H * H_b
    read = weights * H_b + table * H_b
    if case["task"] == "infer":
        return {"bytes": csr + read + states, "flops": rec + leaf}
    grads = 4.0 * weights + (4.0 * case["vocab"] * D if case["vocab"] else 0)
    to_table = leaf * min(1.0, case["vocab"] / leaves) if case["vocab"] else 0.0
    work = {"bytes": read + states + grads + (4.0 * b * H if case["task"] != "train" else 0),
            "flops": 3.0 * rec + 2.0 * leaf + to_table}
    work["bytes"] += csr if case["task"] == "batch" else 8.0 * nodes
    if case["dropout"]:
        work["bytes"] += 4.0 * nodes * H
    if case["task"] == "train":  # labels, losses; Adam reads and writes each weight and both its moments
        trained = weights + case["vocab"] * D + H * case["classes"]
        work["bytes"] += 8.0 * nodes + trained * (24.0 + (2.0 if H_b == 2 else 0.0))
        work["flops"] += 6.0 * nodes * H * case["classes"]
    return work


def tolerance(case):
    """Measured against 64 bits: up to 8e-7 with fp32, and 4e-3 with bf16 (every h is rounded on the way), where two
    passes over the same inputs differ by up to 1.4e-3 (atomic sums in another order)."""
    if case["task"] in ("schedule", "typed"):
        return "exact"
    return {"rel": 1.5e-2} if case["dtype"] == "bf16" else {"rel": 5e-6}


# ---- the same pass in 64 bits ---------------------------------------------------------------------------------

def _order(csr, num_ops):
    """Depths, and the order of the pool: by depth, operation, node."""
    graph_ptr, op, ptr, kids, _ = [x.long() for x in csr]
    n = op.numel()
    parent = torch.repeat_interleave(torch.arange(n, device="cuda"), ptr[1:] - ptr[:-1])
    real = kids >= 0
    parent, child = parent[real], kids[real]
    depth = torch.ones(n, dtype=torch.long, device="cuda")
    while True:
        new = depth.clone().scatter_reduce_(0, parent, depth[child] + 1, "amax")
        if torch.equal(new, depth):
            break
        depth = new
    key = (depth - 1) * num_ops + op
    order = torch.sort(key, stable=True).indices
    pos = torch.empty_like(order)
    pos[order] = torch.arange(n, device="cuda")
    return depth, key, order, pos


def _cell(kind, x, h, c, W_in, W_rec, bias, mask, H):
    """One operation on a block of rows: x the rows read (or None), h and c the children's states."""
    if kind == "embed":
        return x, torch.zeros_like(x)
    if kind == "score":
        e = h[0] @ W_rec[:, 0] + bias
        c0 = torch.zeros_like(h[0])
        return h[0], torch.cat([e[:, None], torch.ones_like(e)[:, None], c0[:, 2:]], 1)
    if kind == "sum":  # the running maximum is held fixed in the gradient
        m = torch.maximum(c[0][:, 0], c[1][:, 0]).detach()
        w = [torch.exp(k[:, 0] - m) for k in c]
        total = w[0] * c[0][:, 1] + w[1] * c[1][:, 1]
        acc = w[0][:, None] * h[0] + w[1][:, None] * h[1]
        return acc, torch.cat([m[:, None], total[:, None], torch.zeros_like(acc)[:, 2:]], 1)
    if kind == "out":
        return h[0] / c[0][:, 1:2], torch.zeros_like(h[0])
    z = bias
    if x is not None:
        z = z + x @ W_in
    if h:
        z = z + torch.cat(h, 1) @ W_rec
    if kind in ("treernn", "proj"):
        t = torch.tanh(z)
        return t, (c[0] if kind == "proj" else torch.zeros_like(t))
    gates = z.split(H, 1)
    i, o, u = torch.sigmoid(gates[0]), torch.sigmoid(gates[-2]), torch.tanh(gates[-1])
    new = i * (u if mask is None else u * mask)
    for k, child in enumerate(c):
        new = new + torch.sigmoid(gates[1 + k]) * child
    return o * torch.tanh(new), new


def _passes(case, d, backward=True):
    """Pools in the order of the schedule and all gradients, in 64 bits; blocks of rows of one depth and operation."""
    H, D, num_ops = case["hidden"], case["in_dim"], len(d["ops"])
    depth, key, order, pos = _order(d["csr"], num_ops)
    ptr, kids, inp = d["csr"][2].long(), d["csr"][3].long(), d["csr"][4].long()
    f = lambda t: None if t is None else t.double()  # noqa: E731
    sets = [{k: f(p[k]) for k in ("W_in", "W_rec", "bias")} for p in d["sets"]]
    table = d["table"]
    n = d["N"]
    h = torch.zeros((n + 1, H), dtype=torch.float64, device="cuda")  # the last row stands for the zero state
    c = torch.zeros_like(h)
    values, rows = torch.unique_consecutive(key[order], return_counts=True)
    blocks, at = [], 0
    for v, r in zip(values.tolist(), rows.tolist()):
        for a in range(at, at + r, 65536):
            blocks.append((v % num_ops, a, min(at + r, a + 65536)))
        at += r
    mask = d.get("mask")

    def block(o, a, b):
        kind, arity, reads, s = d["ops"][o]
        nodes = order[a:b]
        child = []
        for k in range(arity):
            e = kids[ptr[nodes] + k]
            child.append(torch.where(e >= 0, pos[e.clamp(min=0)], torch.full_like(e, n)))
        x = table[inp[nodes]][:, :D].double() if reads else None
        return kind, s, child, x, None if mask is None else mask[a:b, :H].double()

    for o, a, b in blocks:
        kind, s, child, x, m = block(o, a, b)
        h[a:b], c[a:b] = _cell(kind, x, [h[k] for k in child], [c[k] for k in child], sets[s]["W_in"], sets[s]["W_rec"],
                               sets[s]["bias"], m, H)
    if not backward:
        return h[:n], c[:n], order, pos, None
    dh, dc = torch.zeros_like(h), torch.zeros_like(h)
    if "labels" in d:
        loss, dh[:n], head = _head(d, h[:n], order)
    else:
        loss, head = None, None
        has = torch.zeros(n, dtype=torch.bool, device="cuda")
        has[kids[kids >= 0]] = True
        dh[pos[~has]] = d["dh_roots"][:, :H].double()
    grads = [{k: None if t is None else torch.zeros_like(t) for k, t in p.items()} for p in sets]
    d_table = torch.zeros(table.shape, dtype=torch.float64, device="cuda") if case["vocab"] else None
    for o, a, b in reversed(blocks):
        kind, s, child, x, m = block(o, a, b)
        hs = [h[k].requires_grad_() for k in child]
        cs = [c[k].requires_grad_() for k in child]
        if x is not None:
            x.requires_grad_()
        names = [k for k in ("W_in", "W_rec", "bias") if sets[s][k] is not None and kind not in ("embed", "sum", "out")
                 and not (k == "W_in" and x is None) and not (k == "W_rec" and not child)]
        W = {k: sets[s][k].detach().requires_grad_() if k in names else None for k in ("W_in", "W_rec", "bias")}
        with torch.enable_grad():
            out = _cell(kind, x, hs, cs, W["W_in"], W["W_rec"], W["bias"], m, H)
        pairs = [(t, g) for t, g in zip(out, (dh[a:b].clone(), dc[a:b].clone())) if t.requires_grad]
        want = hs + cs + ([x] if x is not None else []) + [W[k] for k in names]
        got = torch.autograd.grad([t for t, _ in pairs], want, [g for _, g in pairs], allow_unused=True)
        for into, at_rows, g in zip([dh] * len(hs) + [dc] * len(cs), child + child, got):
            if g is not None:
                into.index_add_(0, at_rows, g)
        got = got[len(hs) + len(cs):]
        if x is not None:
            if d_table is not None and got[0] is not None:
                d_table[:, :D].index_add_(0, inp[order[a:b]], got[0])
            got = got[1:]
        for k, g in zip(names, got):
            if g is not None:
                grads[s][k] += g
        dh[n].zero_()
        dc[n].zero_()
    return h[:n], c[:n], order, pos, (grads, d_table, loss, head)


def _head(d, h, order):
    """Softmax cross entropy on every node's state, averaged over the nodes."""
    W, b = d["W_cls"].double(), d["b_cls"].double()
    n = h.shape[0]
    z = h @ W + b
    labels = d["labels"].long()[order]
    lse = torch.logsumexp(z, 1)
    loss = torch.empty(n, dtype=torch.float64, device="cuda")
    loss[order] = lse - z.gather(1, labels[:, None])[:, 0]
    dz = torch.exp(z - lse[:, None])
    dz[torch.arange(n, device="cuda"), labels] -= 1.0
    dz = dz / n
    return loss, dz @ W.t(), (h.t() @ dz, dz.sum(0))


def _group_arrays(d, depth, key, order, pos):
    op_arity = torch.tensor([o[1] for o in d["ops"]], device="cuda")
    ptr, kids, inp = d["csr"][2].long(), d["csr"][3].long(), d["csr"][4]
    values, rows = torch.unique_consecutive(key[order], return_counts=True)
    num_ops = len(d["ops"])
    arity = op_arity[d["csr"][1].long()[order]]
    start = torch.cumsum(arity, 0) - arity
    flat = torch.repeat_interleave(ptr[order] - start, arity) + torch.arange(int(arity.sum()), device="cuda")
    e = kids[flat]
    begin = torch.cumsum(rows, 0) - rows
    has = torch.zeros(order.numel(), dtype=torch.bool, device="cuda")
    has[kids[kids >= 0]] = True
    per_level = torch.bincount(depth, minlength=int(depth.max()) + 1)
    got = {"depth": depth, "node_pos": pos, "pos_node": order, "level_ptr": torch.cumsum(per_level, 0),
           "group_level": values // num_ops + 1, "group_op": values % num_ops, "group_row_begin": begin,
           "group_rows": rows, "group_idx_off": start[begin], "child_pos": torch.where(e >= 0, pos[e.clamp(min=0)], e),
           "input_idx": inp.long()[order], "root_pos": pos[~has]}
    return {k: v.to(torch.int32) for k, v in got.items()}


@torch.no_grad()
def exact(case, seed):
    if case["task"] == "typed":
        return None
    d = _inputs(case, seed)
    if case["task"] == "schedule":
        return _group_arrays(d, *_order(d["csr"], len(d["ops"])))
    h, c, order, pos, more = _passes(case, d, case["task"] != "infer")
    kids = d["csr"][3].long()
    has = torch.zeros(d["N"], dtype=torch.bool, device="cuda")
    has[kids[kids >= 0]] = True
    out = {"roots": _padded(h[pos[~has]]), "h": _padded(h), "c": _padded(c)}
    if case["task"] == "infer":
        return out
    grads, d_table, loss, head = more
    flat = []
    for p in grads:
        flat += [p["W_in"], p["W_rec"], p["bias"]]
    if case["task"] == "train":
        return _after_adam(d, loss, out["h"], [g for g in flat if g is not None] + [d_table] + list(head))
    for k, g in enumerate(flat + [d_table]):
        if g is None:
            continue
        if k < len(flat) and d["sets"][k // 3]["kind"] == KIND["score"]:
            if k % 3 == 1:
                room = torch.zeros((g.numel() + 63) // 64 * 64 + 1, dtype=torch.float64, device="cuda")
                room[:g.numel()], room[-1] = g.reshape(-1), flat[k + 1][0]
                out["d%d" % k] = room
            continue
        out["d%d" % k] = g
    return out


def _after_adam(d, loss, h, grads):
    weights = []
    for p in d["sets"]:
        weights += [p[k].double() for k in ("W_in", "W_rec", "bias") if p[k] is not None]
    weights += [d["table"].double(), d["W_cls"].double(), d["b_cls"].double()]
    lr = 1e-3 * math.sqrt(1 - 0.999) / (1 - 0.9)  # the first step's
    new = [w - lr * (0.1 * g) / (torch.sqrt(0.001 * g * g) + 1e-8) for w, g in zip(weights, grads)]
    return {"loss": loss, "h": h, "weights": new, "grads": grads}
