"""Backward passes that ask for no node gradients skip the ones nobody reads (cell-state gradients of operations without a
cell state, everything below a level of embeddings): the parameters' gradients against the oracle, with and without the
leaf table's, the gradient rows filled with NaN before, so that a row read after all shows."""
import numpy as np
import pytest

from paper_1702_02181_amd import gen
from tests import gpu_common as C

pytestmark = pytest.mark.gpu


def _embed_under(kinds, hidden, dtype, seed=4):
    """Graphs over embeddings: chains of the unary kinds, random trees of the binary one, some leaves directly below
    high nodes, and a zero state."""
    rng = np.random.default_rng(seed)
    ops = [gen.OpSpec(gen.KIND_EMBED, 0, 1, 0)]
    params = [gen.make_param_set(rng, gen.KIND_EMBED, hidden, 0, hidden, dtype)]
    for k in kinds:
        arity = 1 if k in (gen.KIND_PROJ, gen.KIND_LSTM) else 2
        ops.append(gen.OpSpec(k, arity, 0, len(params)))
        params.append(gen.make_param_set(rng, k, 0, arity, hidden, dtype))
    graphs = []
    for _ in range(30):
        b = gen._GraphBuilder()
        nodes = [b.add(0, (), int(rng.integers(0, 20))) for _ in range(4)]
        for _ in range(8):
            o = int(rng.integers(1, len(ops)))
            kids = [int(rng.choice(nodes[-3:] + nodes[:2])) for _ in range(ops[o].arity)]
            if rng.random() < 0.1:
                kids[-1] = -1
            nodes.append(b.add(o, kids))
        graphs.append(b.arrays())
    table = gen._finish_values(rng.standard_normal((20, hidden)), dtype)
    return gen._finish("embed", dtype, hidden, gen.assemble(graphs), ops, params, table, rng, True)


WORKLOADS = {
    "proj": lambda d: _embed_under([gen.KIND_PROJ], 40, d),
    "treernn": lambda d: _embed_under([gen.KIND_TREERNN], 40, d),
    "proj+treernn": lambda d: _embed_under([gen.KIND_PROJ, gen.KIND_TREERNN], 40, d),
    "proj+treelstm": lambda d: _embed_under([gen.KIND_PROJ, gen.KIND_TREELSTM], 40, d),
    "lstm+proj+treernn": lambda d: _embed_under([gen.KIND_LSTM, gen.KIND_PROJ, gen.KIND_TREERNN], 40, d),
    "attention": lambda d: gen.attention(num_graphs=9, length=(1, 12), hidden=96, dtype=d),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("table_grad", [False, True])
@pytest.mark.parametrize("name", sorted(WORKLOADS))
def test_parameter_gradients(name, table_grad, dtype):
    import torch
    from oracle import compare
    from paper_1702_02181_amd.runner import DeviceRun
    w = WORKLOADS[name](dtype)
    o = C.run_oracle(w, table_grad=table_grad)
    dev = DeviceRun(w)
    dev.forward()
    fwd = dev.fwd_bytes
    dev.ws[fwd:].view(torch.uint8).fill_(255)  # every float past the saved activations is NaN
    dev.alloc_grads(table_grad)
    dev.set_upstream(w.dh_roots)
    dev.backward()
    grads, d_table = dev.weight_grads()
    tol = C.TOL[dtype]
    for k, (g, r) in enumerate(zip(grads, o["grads"])):
        for key in ("W_in", "W_rec", "bias"):
            if g[key] is None or r[key] is None:
                continue
            if w.params[k].kind == gen.KIND_ATTN_SCORE and key == "bias":
                continue  # zero up to rounding: the softmax ignores a common shift of the scores
            err = compare.rel_err(g[key].reshape(1, -1), np.asarray(r[key]).reshape(1, -1))
            assert err <= tol, (k, key, err)
    if table_grad:
        assert compare.rel_err(d_table.reshape(1, -1), np.asarray(o["d_table"]).reshape(1, -1)) <= tol
