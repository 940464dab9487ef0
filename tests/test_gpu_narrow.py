"""Levels on 16-row tiles against the oracle, forward and backward: every internal level has exactly `rows` rows, at the
edges of the row tiles (16, 32), of the sizes that choose single or double row tiles and 4, 8 or 16 hidden units per
workgroup, and one row past them."""
import numpy as np
import pytest

from paper_1702_02181_amd import gen
from tests import gpu_common as C

pytestmark = pytest.mark.gpu


def _levels(rows, hidden, dtype, mixed, seed=3):
    """`rows` graphs with two internal levels each: a Tree-LSTM spine, or (mixed) LSTM, Tree-LSTM and PROJ at each depth."""
    rng = np.random.default_rng(seed)
    graphs = []
    for i in range(rows):
        b = gen._GraphBuilder()
        if mixed:
            gen.lstm_chain_reduce(b, 1 + i % 4, rng, 4 * i, 0.5, 0, 1, 2)
        else:
            gen.caterpillar(b, 2, 0, 1, range(3 * i, 3 * i + 3))
        graphs.append(b.arrays())
    csr = gen.assemble(graphs)
    D = 40
    table = gen._finish_values(rng.standard_normal((4 * rows, D)), dtype)
    if mixed:
        ops = [gen.OpSpec(gen.KIND_LSTM, 1, 1, 0), gen.OpSpec(gen.KIND_TREELSTM, 2, 0, 1), gen.OpSpec(gen.KIND_PROJ, 1, 0, 2)]
        params = [gen.make_param_set(rng, gen.KIND_LSTM, D, 1, hidden, dtype),
                  gen.make_param_set(rng, gen.KIND_TREELSTM, 0, 2, hidden, dtype),
                  gen.make_param_set(rng, gen.KIND_PROJ, 0, 1, hidden, dtype)]
    else:
        ops = [gen.OpSpec(gen.KIND_TREELSTM, 0, 1, 0), gen.OpSpec(gen.KIND_TREELSTM, 2, 0, 0)]
        params = [gen.make_param_set(rng, gen.KIND_TREELSTM, D, 2, hidden, dtype)]
    return gen._finish("narrow", dtype, hidden, csr, ops, params, table, rng, True)


@pytest.mark.parametrize("dtype,hidden,rows,mixed", [
    ("f32", 40, 17, False), ("f32", 300, 16, False), ("f32", 300, 64, False), ("f32", 300, 65, False),
    ("f32", 256, 100, False), ("f32", 200, 300, False), ("f32", 130, 33, True),
    ("bf16", 1, 1, False), ("bf16", 300, 48, False), ("bf16", 300, 49, False), ("bf16", 300, 130, False),
    ("bf16", 256, 257, False), ("bf16", 64, 90, True), ("bf16", 512, 31, True),
])
def test_narrow_levels(dtype, hidden, rows, mixed):
    w = _levels(rows, hidden, dtype, mixed)
    errs = C.compare_all(w, C.run_device(w), C.run_oracle(w))
    print(dtype, hidden, rows, mixed, errs)


@pytest.mark.parametrize("dtype,hidden,rows,mixed", [
    ("f32", 1024, 33, False), ("f32", 768, 128, False), ("f32", 700, 65, True),
    ("bf16", 1024, 64, False), ("bf16", 768, 128, False), ("bf16", 1024, 40, True), ("bf16", 1100, 20, False),
])
def test_narrow_levels_of_wide_states(dtype, hidden, rows, mixed):
    """The same for states wider than 512: single and double row tiles of 4 to 16 units, and a width past the forward's
    limit whose dz . W^T alone is narrow."""
    w = _levels(rows, hidden, dtype, mixed)
    errs = C.compare_all(w, C.run_device(w), C.run_oracle(w))
    print(dtype, hidden, rows, mixed, errs)
