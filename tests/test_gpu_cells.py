"""GPU forward / backward parity against the fp64 oracle, through the C ABI.

Sizes are ones the oracle finishes in seconds while still spanning several
workgroup tiles and ragged tails (row counts that are not multiples of the
tile heights, hidden sizes that are not multiples of 64)."""
import numpy as np
import pytest

from paper_1702_02181_amd import gen
from tests import gpu_common as C

pytestmark = pytest.mark.gpu


def test_config1_full_forward_fp32():
    w = gen.config1()
    g, o = C.run_device(w), C.run_oracle(w)
    C.compare_all(w, g, o)


def test_config1_backward_with_table_grad():
    w = gen.config1()
    w.backward = True
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)


@pytest.mark.parametrize("leaves,graphs", [(64, 4), (37, 5)])
def test_config2_shape_fp32_fwd_bwd(leaves, graphs):
    w = gen.config2(num_graphs=graphs, leaves=leaves)
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)


def test_config2_per_node_upstream_gradients():
    w = gen.config2(num_graphs=3, leaves=24)
    dh = np.random.default_rng(5).standard_normal((w.num_nodes, w.hidden))
    g, o = C.run_device(w, dh_nodes=dh), C.run_oracle(w, dh_nodes=dh)
    C.compare_all(w, g, o)


@pytest.mark.parametrize("cfg", [2, 3])
def test_leaf_forget_columns_of_w_in_get_exactly_zero(cfg):
    """Tree-LSTM leaves have zero child states, so the forget-gate columns of W_in receive exactly zero
    gradient (internal nodes of these workloads read no input). The leaf kernels skip those gates entirely:
    the columns must stay at the caller's zeros, bit for bit, while the live columns match the oracle."""
    w = gen.config2(num_graphs=3, leaves=24) if cfg == 2 else gen.config3(num_graphs=8)
    g, o = C.run_device(w, table_grad=(cfg == 3)), C.run_oracle(w, table_grad=(cfg == 3))
    H = w.hidden
    dW = g["grads"][0]["W_in"]
    assert np.all(dW[:, H:3 * H] == 0)
    assert np.all(o["grads"][0]["W_in"][:, H:3 * H] == 0)
    C.compare_all(w, g, o, table_grad=(cfg == 3))


def test_config3_shape_bf16_h300():
    w = gen.config3(num_graphs=24)
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)


def test_config4_shape_mixed_ops_bf16():
    w = gen.config4(num_graphs=10, max_chain=40)
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)


def test_config5_shape_dag_bf16():
    w = gen.config5(num_graphs=6, hidden=256, vocab=300, spine_range=(60, 200), balanced_leaves=64)
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)


def test_batching_invariance_on_gpu():
    """Each graph's forward states inside the batch equal, bit for bit, those of the graph scheduled alone and
    those of the batch with its graphs in reverse order; and the batch matches the oracle.  Every level here
    has at most 128 rows, so alone and in the batch each level sums K in the same order, and a row's arithmetic
    does not depend on the rows around it: batching is a pure rewrite (Section 2).  (test_gpu_batch_invariance.py
    has the widths and row counts at which the tiles change.)"""
    w = gen.config4(num_graphs=6, max_chain=20, hidden=64, in_dim=32)
    g = C.run_device(w, backward=False)
    assert max(np.diff(g["sched"]["level_ptr"])) <= 128
    C.compare_all(w, g, C.run_oracle(w, backward=False), check_backward=False)
    gp = w.graph_ptr
    for k in (0, 3, 5):
        gk = C.run_device(gen.subset(w, [k]), backward=False)
        assert np.array_equal(gk["h"], g["h"][gp[k]:gp[k + 1]]), k
        assert np.array_equal(gk["c"], g["c"][gp[k]:gp[k + 1]]), k
    order = list(range(w.num_graphs))[::-1]
    wr = gen.subset(w, order)
    gr = C.run_device(wr, backward=False)
    gpr = wr.graph_ptr
    for i, k in enumerate(order):
        assert np.array_equal(gr["h"][gpr[i]:gpr[i + 1]], g["h"][gp[k]:gp[k + 1]]), k


@pytest.mark.parametrize("mode", ["manual", "dynamic", "full"])
def test_table1_workloads_forward(mode):
    """The three schedules of the Table 1 protocol (one group per tree node; per (depth, op); random shapes)
    compute the fp64 oracle's states of the same trees (fp32, H = 1024 as in the table)."""
    w = gen.table1(3, mode, hidden=1024, vocab=200)
    g, o = C.run_device(w), C.run_oracle(w)
    C.compare_all(w, g, o)


@pytest.mark.parametrize("case", ["cfg4_bf16", "random_f32", "table1_manual"])
def test_level_launches_match_one_launch_per_group(case):
    """Levels of several operations run their narrow groups as level launches (one launch for the level's
    contractions, one for its K-split epilogues, one for its cell backwards, one for its dz . W^T).  The
    forward states equal those of one launch per group (fold_level_launches(0)) bit for bit -- at these sizes
    every group sums K in the same order either way (always so up to 128 rows and H = 1,024) -- and the gradients up
    to the order of atomic additions; both match the oracle."""
    from oracle import compare
    from paper_1702_02181_amd import fold as F
    from tests.test_gpu_random import _random_batch
    if case == "cfg4_bf16":
        w = gen.config4(num_graphs=12, max_chain=40, hidden=256, in_dim=64)
    elif case == "random_f32":
        w = _random_batch(77, 64, "f32", n_graphs=40)
    else:
        w = gen.table1(16, "manual", hidden=128, vocab=100)
    table_grad = w.backward
    prev = F.fold_level_launches(True)
    try:
        merged = C.run_device(w, table_grad=table_grad)
        F.fold_level_launches(False)
        single = C.run_device(w, table_grad=table_grad)
    finally:
        F.fold_level_launches(prev)
    for k in ("h", "c", "roots"):
        assert np.array_equal(merged[k], single[k]), k
    if w.backward:
        # atomic adds in another order move fp32 sums by ulps; with bf16 parameters such a move can flip the
        # bf16 rounding of a dz element, and the flip propagates down the levels (here ~1e-3 after 40 levels)
        tol = {"f32": 1e-6, "bf16": 1e-2}[w.dtype]
        for k in ("dh", "dc"):
            assert compare.rel_err(merged[k], single[k]) <= tol, k
    C.compare_all(w, merged, C.run_oracle(w, table_grad=table_grad), table_grad=table_grad)


def test_backward_rejects_misaligned_gradient_buffers():
    """The backward's gradient rows are accessed 16 bytes at a time: dh_roots, dh_nodes, dh_out, dc_out and the
    workspace must be 16-byte aligned, anything else is FOLD_E_INVALID before any work is queued."""
    import torch
    from paper_1702_02181_amd import fold as F
    from paper_1702_02181_amd.runner import DeviceRun
    w = gen.config2(num_graphs=2, leaves=8)
    dev = DeviceRun(w, with_backward=True)
    dev.forward()
    dev.alloc_grads(False)
    dev.set_upstream(w.dh_roots, None)
    good = torch.zeros((dev.N + 1) * dev.ld, dtype=torch.float32, device="cuda")
    bad = good[1:]  # 4 bytes past a 256-byte boundary
    roots_bad = torch.zeros(dev.R * dev.ld + 1, dtype=torch.float32, device="cuda")[1:]
    ws_bad = torch.empty(dev.ws_bytes + 16, dtype=torch.uint8, device="cuda")[8:]
    cases = [dict(dh_out=bad), dict(dc_out=bad), dict(dh_nodes=bad), dict(dh_roots=roots_bad), dict(ws=ws_bad)]
    for case in cases:
        args = dict(dh_roots=dev.dh_roots, dh_nodes=None, dh_out=None, dc_out=None, ws=dev.ws)
        args.update(case)
        with pytest.raises(F.FoldError) as e:
            F.fold_backward(dev.sched.handle, dev.packed.handle, dev.table, dev.leaf_rows, dev.h_pool, dev.c_pool,
                            args["dh_roots"], args["dh_nodes"], dev.grads, args["dh_out"], args["dc_out"], args["ws"],
                            dev.ws_bytes, dev.stream)
        assert e.value.code == F.FOLD_E_INVALID and "aligned" in str(e.value), list(case)
    torch.cuda.synchronize()


def _table_runs_case(dtype, graphs=256, leaves=64, H=32, V=5, seed=21, distinct=False):
    """Balanced trees of `leaves` Tree-LSTM leaves with an LSTM chain of three steps on each root; every leaf
    and LSTM step reads one of V leaf-table rows, row 0 for 80 % of them (distinct: a table row of its own)."""
    from tests._helpers import make_workload
    rng = np.random.default_rng(seed)
    if distinct:
        V = graphs * (leaves + 3)
    ops = [gen.OpSpec(gen.KIND_TREELSTM, 0, 1, 0), gen.OpSpec(gen.KIND_TREELSTM, 2, 0, 0),
           gen.OpSpec(gen.KIND_LSTM, 1, 1, 1)]
    params = [gen.make_param_set(rng, gen.KIND_TREELSTM, H, 2, H, dtype),
              gen.make_param_set(rng, gen.KIND_LSTM, H, 1, H, dtype)]
    table = gen._finish_values(0.1 * rng.standard_normal((V, H)), dtype)

    rows = iter(rng.permutation(V).tolist())

    def token():
        if distinct:
            return next(rows)
        return 0 if rng.random() < 0.8 else int(rng.integers(1, V))
    batch = []
    for _ in range(graphs):
        nodes = [(0, [], token()) for _ in range(leaves)]
        level = list(range(leaves))
        while len(level) > 1:
            nxt = []
            for a, b in zip(level[0::2], level[1::2]):
                nodes.append((1, [a, b], -1))
                nxt.append(len(nodes) - 1)
            level = nxt
        for _ in range(3):
            nodes.append((2, [len(nodes) - 1], token()))
        batch.append(nodes)
    w = make_workload(batch, ops, params, H, table, dtype=dtype, seed=seed, name=f"table_runs_{dtype}")
    w.backward = True
    return w


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_leaf_table_gradient_long_runs(dtype):
    """The leaf-table gradient sums dz over the rows of each (op, leaf-table row) before contracting once per
    distinct leaf-table row.  16,384 leaves and 768 LSTM steps read 5 table rows (row 0 for 80 % of them): runs
    of thousands of rows cross many summing workgroups (whose partial sums are added atomically), and two ops
    add into the same table rows.  Every state and gradient against the oracle, the table gradient included."""
    w = _table_runs_case(dtype)
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)
    # and row by row (the table's rows differ in size: row 0 sums 80 % of the rows)
    from oracle import compare
    assert compare.rel_err(g["d_table"], o["d_table"]) <= C.TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_leaf_table_gradient_distinct_rows(dtype):
    """Every leaf and LSTM step reads a table row of its own (37 graphs: 592 leaves and 111 steps, neither a
    multiple of 64), so every row is a run of its own and the scheduler's per-operation run counts, added once
    per operation and wave, meet an operation boundary inside a wave.  Table gradient row by row against the
    oracle, every other state and gradient too."""
    w = _table_runs_case(dtype, graphs=37, leaves=16, distinct=True)
    g, o = C.run_device(w, table_grad=True), C.run_oracle(w, table_grad=True)
    C.compare_all(w, g, o, table_grad=True)
    from oracle import compare
    assert compare.rel_err(g["d_table"], o["d_table"]) <= C.TOL[dtype]
