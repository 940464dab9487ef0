"""The scheduler at the edges of its tiles and digits, bit-exact against the oracle's reference scheduler: batches one
node around a tile of 2,048 and around the 32 tiles up to which a tile adds up its predecessors itself, keys of one, two
and three 10-bit digits, and the leaf-table runs of several operations over many tiles (through the gradient they sum)."""
import numpy as np
import pytest

from paper_1702_02181_amd import gen
from tests import gpu_common as C
from tests.test_gpu_schedule import _gpu_sched

pytestmark = pytest.mark.gpu


def _chains(rng, total, longest, num_ops):
    """`total` nodes in chains of up to `longest`: an embedding, then random unary operations."""
    graphs, left = [], total
    while left:
        n = min(left, int(rng.integers(1, longest + 1)))
        op = np.concatenate([[0], rng.integers(1, num_ops, n - 1)]).astype(np.int32)
        cnt = np.concatenate([[0], np.ones(n - 1)]).astype(np.int32)
        inp = np.concatenate([[int(rng.integers(0, 9))], -np.ones(n - 1)]).astype(np.int64)
        graphs.append((op, cnt, np.arange(n - 1), inp))
        left -= n
    ops = [gen.OpSpec(gen.KIND_EMBED, 0, 1, 0)] + [gen.OpSpec(gen.KIND_PROJ, 1, 0, 1)] * (num_ops - 1)
    csr = gen.assemble(graphs)
    return gen.Workload("chains", "f32", 2, ops=ops, params=[], leaf_table=np.zeros((9, 2), np.float32),
                        dh_roots=np.zeros((len(graphs), 2), np.float32), **csr)


@pytest.mark.parametrize("total,longest,num_ops", [
    (1, 1, 2), (63, 5, 2), (4096, 4000, 3), (4096, 9, 256), (4097, 9, 5),  # one launch up to 4,096 nodes
    (2047, 9, 3), (2048, 9, 2), (2049, 40, 5),
    (65535, 30, 2), (65537, 30, 4),     # 32 tiles and one node more: the column scan
    (3000, 700, 3),                     # two digits
    (5000, 5000, 256),                  # one chain of 5,000: keys past 2^20, three digits, no room in LDS
])
def test_tile_and_digit_edges(total, longest, num_ops):
    w = _chains(np.random.default_rng(total + num_ops), total, longest, num_ops)
    C.assert_schedule_equal(_gpu_sched(w), C.oracle_schedule(w))


def test_dags_of_both_paths():
    """Shared children, a child taken twice and zero states, just below and above the one-launch limit."""
    from tests.test_oracle_schedule import random_dag
    for seed, n in ((5, 130), (6, 420)):
        w = random_dag(np.random.default_rng(seed), n_graphs=n, max_nodes=60)
        C.assert_schedule_equal(_gpu_sched(w), C.oracle_schedule(w))


@pytest.mark.parametrize("total", [200, 6000])
@pytest.mark.parametrize("what", ["op", "arity", "child", "other graph", "input", "cycle", "pointers", "lowest"])
def test_errors_of_both_paths(total, what):
    """Every error code from the one-launch schedule and from the tiled one; the lowest node counts."""
    from paper_1702_02181_amd import fold as F
    w = _chains(np.random.default_rng(1), total, 12, 3)
    gp, at = w.graph_ptr, int(np.nonzero(np.diff(w.graph_ptr) > 4)[0][3])  # a graph of five nodes or more
    first = int(gp[at])
    edge = lambda v: int(w.child_ptr[v])  # noqa: E731
    code = {"op": F.FOLD_E_OP, "arity": F.FOLD_E_ARITY, "child": F.FOLD_E_CHILD, "other graph": F.FOLD_E_CHILD,
            "input": F.FOLD_E_INPUT, "cycle": F.FOLD_E_CYCLE, "pointers": F.FOLD_E_INVALID, "lowest": F.FOLD_E_INPUT}[what]
    if what == "op":
        w.node_op[first + 2] = 3
    elif what == "arity":
        w.node_op[first + 2], w.node_input[first + 2] = 0, 0
    elif what == "child":
        w.child_idx[edge(first + 2)] = total
    elif what == "other graph":
        w.child_idx[edge(first + 2)] = first - 1
    elif what == "input":
        w.node_input[first] = 9
    elif what == "cycle":
        w.child_idx[edge(first + 1)] = first + 3
    elif what == "pointers":
        w.child_ptr[first + 2] = w.child_ptr[-1] + 1
    else:  # a cycle and an operation out of range come after a bad input in node order
        w.node_input[first] = -1
        w.node_op[first + 3] = 7
        w.child_idx[edge(first + 1)] = first + 2
    with pytest.raises(F.FoldError) as e:
        _gpu_sched(w)
    assert e.value.code == code
    if what == "cycle":
        assert f"(node {first})" in str(e.value)
    elif what == "lowest":
        assert f"(node {first})" in str(e.value)


@pytest.mark.parametrize("total,rows", [(1, 1), (2049, 1), (4096, 3000), (4097, 3000), (70001, 5), (70001, 100003)])
def test_leaf_table_runs(total, rows):
    """Nodes that are embeddings of two operations, both reading random rows: each leaf-table row's gradient is the sum
    of its nodes' upstream gradients (fp32 sums of n terms: error below n 2^-24 times the sum of their magnitudes)."""
    import torch
    from paper_1702_02181_amd.runner import DeviceRun
    rng = np.random.default_rng(total + rows)
    op, inp = rng.integers(0, 2, total), rng.integers(0, rows, total)
    csr = dict(graph_ptr=np.arange(total + 1, dtype=np.int32), node_op=op.astype(np.int32),
               child_ptr=np.zeros(total + 1, np.int32), child_idx=np.zeros(0, np.int32), node_input=inp.astype(np.int32))
    params = [gen.ParamSet(gen.KIND_EMBED, 2, 0, None, None, np.zeros(0, np.float32))] * 2
    w = gen.Workload("rows", "f32", 2, ops=[gen.OpSpec(gen.KIND_EMBED, 0, 1, 0), gen.OpSpec(gen.KIND_EMBED, 0, 1, 1)],
                     params=params, leaf_table=np.zeros((rows, 2), np.float32),
                     dh_roots=rng.standard_normal((total, 2)).astype(np.float32), **csr)
    dev = DeviceRun(w)
    dev.forward()
    dev.alloc_grads(True)
    dev.set_upstream(w.dh_roots)
    dev.backward()
    torch.cuda.synchronize()
    got = dev.d_table.cpu().numpy()[:, :2].astype(np.float64)
    want, size, count = np.zeros((rows, 2)), np.zeros((rows, 2)), np.bincount(inp, minlength=rows)[:, None]
    np.add.at(want, inp, w.dh_roots.astype(np.float64))
    np.add.at(size, inp, np.abs(w.dh_roots.astype(np.float64)))
    assert np.all(np.abs(got - want) <= (count + 1) * 2.0 ** -24 * size)


def test_schedules_from_several_threads():
    """Schedules made and freed by four threads on streams of their own: the blocks they hand one another are whole."""
    import threading
    import torch
    works = [_chains(np.random.default_rng(k), 500 + 700 * k, 12, 3) for k in range(4)]
    refs = [C.oracle_schedule(w) for w in works]
    failed = []

    def go(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(6):
                    C.assert_schedule_equal(_gpu_sched(works[(k + i) % 4]), refs[(k + i) % 4])
        except BaseException as e:  # noqa: BLE001 -- reported by the main thread
            failed.append(repr(e))

    threads = [threading.Thread(target=go, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_schedule_freed_while_another_thread_captures():
    """A schedule freed by one thread while another records a stream: the recording ends well and replays, and a schedule
    made afterwards is whole."""
    import threading
    import torch
    from paper_1702_02181_amd import fold as F
    w = _chains(np.random.default_rng(3), 700, 12, 3)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    sched = F.Schedule(i32(w.graph_ptr), i32(w.node_op), i32(w.child_ptr), i32(w.child_idx), i32(w.node_input),
                       [(o.kind, o.arity, o.has_input, o.param_set) for o in w.ops], w.leaf_table.shape[0])
    x, y = torch.arange(64, dtype=torch.float32, device="cuda"), torch.zeros(64, device="cuda")
    torch.cuda.synchronize()

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        torch.mul(x, 2, out=y)
        t = threading.Thread(target=sched.__del__)
        t.start()
        t.join()
    assert sched.handle is None
    for k in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, 2 * x), k
        C.assert_schedule_equal(_gpu_sched(w), C.oracle_schedule(w))
