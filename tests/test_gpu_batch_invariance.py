"""A graph's forward states have the same bits alone and in a batch whose levels stay at 128 rows, for every width: the
sums over K must not be taken in another order because a level got more rows or another operation beside it.  The batches
have levels on both sides of the sizes at which the tiles change (16, 32, 48, 64 and 96 rows)."""
import numpy as np
import pytest

from paper_1702_02181_amd import fold as F
from paper_1702_02181_amd import gen
from tests import gpu_common as C

pytestmark = pytest.mark.gpu

D = 24
OPS = {"treelstm": [gen.OpSpec(gen.KIND_TREELSTM, 0, 1, 0), gen.OpSpec(gen.KIND_TREELSTM, 2, 0, 0)],
       "lstm": [gen.OpSpec(gen.KIND_LSTM, 1, 1, 0)],
       "lstm+treelstm": [gen.OpSpec(gen.KIND_TREELSTM, 0, 1, 0), gen.OpSpec(gen.KIND_TREELSTM, 2, 0, 0),
                         gen.OpSpec(gen.KIND_LSTM, 1, 1, 1)]}


def _chains(model, counts, hidden, dtype):
    """counts[k] graphs of kind k, each with one node on every one of four levels: Tree-LSTM nodes over a leaf (both
    children the node below), or an LSTM chain."""
    rng = np.random.default_rng(hidden)
    ops = OPS[model]
    graphs = []
    for k, n in enumerate(counts):
        lstm = ops[-1].kind == gen.KIND_LSTM and k == len(counts) - 1
        for _ in range(n):
            b = gen._GraphBuilder()
            cur = -1 if lstm else b.add(0, (), int(rng.integers(0, 50)))
            for _ in range(4 if lstm else 3):
                if lstm:
                    cur = b.add(len(ops) - 1, (cur,), int(rng.integers(0, 50)))
                else:
                    cur = b.add(1, (cur, cur))
            graphs.append(b.arrays())
    table = gen._finish_values(rng.standard_normal((50, D)), dtype)
    sets = {o.param_set: o.kind for o in ops}
    params = [gen.make_param_set(rng, kind, D, 2 if kind == gen.KIND_TREELSTM else 1, hidden, dtype)
              for _, kind in sorted(sets.items())]
    return gen._finish("chains", dtype, hidden, gen.assemble(graphs), ops, params, table, rng, False)


def _same(w, whole, graphs):
    part = C.run_device(gen.subset(w, graphs), backward=False)
    at = np.concatenate([np.arange(w.graph_ptr[g], w.graph_ptr[g + 1]) for g in graphs])
    for k in ("h", "c"):
        assert np.array_equal(part[k], whole[k][at]), (k, len(graphs), int((part[k] != whole[k][at]).sum()))


# widths of one operation: the whole range; several operations on a level: up to 1,024
@pytest.mark.parametrize("model,dtype,hidden", [
    ("treelstm", "f32", 300), ("treelstm", "f32", 512), ("treelstm", "f32", 1024), ("treelstm", "f32", 2048),
    ("lstm", "f32", 700), ("treelstm", "bf16", 300), ("treelstm", "bf16", 1024), ("treelstm", "bf16", 1100),
    ("treelstm", "bf16", 2048), ("lstm", "bf16", 4096),
])
def test_levels_of_up_to_128_rows(model, dtype, hidden):
    w = _chains(model, [128], hidden, dtype)
    whole = C.run_device(w, backward=False)
    assert max(np.diff(whole["sched"]["level_ptr"])) <= 128
    for n in (1, 16, 17, 40, 49, 64, 65, 97):
        _same(w, whole, list(range(n)))
    few = gen.subset(w, [0, 1, 2])
    C.compare_all(few, C.run_device(few, backward=False), C.run_oracle(few, backward=False), check_backward=False)


@pytest.mark.parametrize("dtype,hidden,counts", [("f32", 512, (70, 10)), ("f32", 300, (5, 100)), ("f32", 1024, (64, 64)),
                                                 ("bf16", 512, (90, 30)), ("bf16", 1024, (100, 28))])
def test_levels_of_two_operations(dtype, hidden, counts):
    """The same with an LSTM and a Tree-LSTM on every level, against each alone, and without level launches."""
    w = _chains("lstm+treelstm", counts, hidden, dtype)
    whole = C.run_device(w, backward=False)
    assert max(np.diff(whole["sched"]["level_ptr"])) <= 128
    a, b = counts
    for graphs in ([0], [a], list(range(a)), list(range(a, a + b)), [0, 1, a, a + 1, a + 2]):
        _same(w, whole, graphs)
    prev = F.fold_level_launches(False)
    try:
        single = C.run_device(w, backward=False)
    finally:
        F.fold_level_launches(prev)
    for k in ("h", "c", "roots"):
        assert np.array_equal(whole[k], single[k]), k


@pytest.mark.parametrize("dtype,hidden,counts", [("f32", 512, (70, 100)), ("bf16", 512, (256, 256))])
def test_merged_and_single_above_128_rows(dtype, hidden, counts):
    """Above 128 rows a group can run on other tiles beside another one than alone (the 70 rows; 512 workgroups together):
    the order of the sums may then differ, the states match the oracle either way."""
    w = _chains("lstm+treelstm", counts, hidden, dtype)
    o = C.run_oracle(w, backward=False)
    prev = F.fold_level_launches(True)
    try:
        for on in (True, False):
            F.fold_level_launches(on)
            C.compare_all(w, C.run_device(w, backward=False), o, check_backward=False)
    finally:
        F.fold_level_launches(prev)
