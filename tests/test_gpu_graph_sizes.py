"""The depth walk with each of its workgroup sizes (chosen by the nodes of an average graph: below 16, below 1,024, above),
on graphs that fit the LDS and graphs that do not, alone and among small ones: every schedule array against the oracle."""
import numpy as np
import pytest

from oracle import paper_schedule as PS
from paper_1702_02181_amd import gen
from tests import gpu_common as C
from tests.test_gpu_paper_schedule import _assert_equal, _gpu
from tests.test_gpu_schedule import _gpu_sched
from tests.typed_graphs import tree_lstm_paper_form

pytestmark = pytest.mark.gpu


def _graph(rng, n, reach):
    """n nodes: embeddings, and operations on two of the `reach` nodes before them (shared, taken twice, or a zero state)."""
    op = (rng.random(n) < 0.6).astype(np.int32)
    op[0] = 0
    v = np.repeat(np.nonzero(op)[0], 2)
    kids = v - 1 - (rng.random(v.size) * np.minimum(v, reach)).astype(np.int64)
    kids[rng.random(v.size) < 0.02] = -1
    return op, 2 * op, kids, np.where(op == 1, -1, rng.integers(0, 9, n))


@pytest.mark.parametrize("sizes,reach", [
    ([5000], 40), ([30000], 30000), ([1500] * 6, 1500),         # 1,024 threads: scratch memory, and LDS
    ([980, 1000, 1020, 1100, 2000], 20), ([20] * 300 + [6000], 50),  # 256
    ([3] * 2000 + [5000], 3000), ([1] * 5000, 1),                # 128
    ([0, 0, 4500, 0], 500),
])
def test_graph_sizes(sizes, reach):
    rng = np.random.default_rng(len(sizes) + sizes[-1])
    graphs = [_graph(rng, n, reach) if n else tuple(np.zeros(0, np.int64) for _ in range(4)) for n in sizes]
    csr = gen.assemble(graphs)
    ops = [gen.OpSpec(gen.KIND_EMBED, 0, 1, 0), gen.OpSpec(gen.KIND_TREERNN, 2, 0, 1)]
    w = gen.Workload("sizes", "f32", 2, ops=ops, params=[], leaf_table=np.zeros((9, 2), np.float32),
                     dh_roots=np.zeros((0, 2), np.float32), **csr)
    C.assert_schedule_equal(_gpu_sched(w), C.oracle_schedule(w))


@pytest.mark.parametrize("graphs,leaves", [(2, 700), (1, 2500), (8, 40), (30, 3)])
def test_typed_graph_sizes(graphs, leaves):
    w = gen.config2(num_graphs=graphs, leaves=leaves, hidden=2)
    (gp, *g), ops, T = tree_lstm_paper_form(w)
    _assert_equal(_gpu(gp, g, ops, T), PS.paper_schedule(*g, ops, T), g, T)
