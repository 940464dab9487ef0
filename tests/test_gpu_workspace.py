"""The forward's workspace holds partial sums only for levels that write them: batches whose levels all run on narrow tiles
need the saved activations alone, and a forward of levels of both sorts stays inside what fold_workspace_size asks for,
with and without level launches."""
import numpy as np
import pytest

from paper_1702_02181_amd import fold as F
from paper_1702_02181_amd.runner import DeviceRun
from tests.test_gpu_batch_invariance import _chains
from tests.test_gpu_narrow import _levels

pytestmark = pytest.mark.gpu


def _sizes(w):
    dev = DeviceRun(w, with_backward=False)
    gmax = max({0: 5, 1: 4}[0 if o.kind == 2 else 1] for o in w.ops)  # Tree-LSTM, or LSTM alone
    hp = (w.hidden + 63) // 64 * 64
    return dev, w.num_nodes * gmax * hp * (2 if w.dtype == "bf16" else 4)


@pytest.mark.parametrize("model,dtype,hidden,counts", [
    ("treelstm", "f32", 1024, [64]), ("treelstm", "f32", 1024, [128]), ("lstm+treelstm", "f32", 512, [70, 10]),
    ("lstm+treelstm", "bf16", 512, [60, 60]), ("treelstm", "bf16", 300, [100]),
])
def test_narrow_levels_need_no_partial_sums(model, dtype, hidden, counts):
    dev, saved = _sizes(_chains(model, counts, hidden, dtype))
    assert dev.fwd_bytes == (saved + 255) // 256 * 256


@pytest.mark.parametrize("dtype,hidden,rows,mixed", [("f32", 320, 300, False), ("f32", 400, 400, True),
                                                     ("bf16", 512, 500, True), ("bf16", 300, 330, True)])
def test_forward_stays_inside_its_workspace(dtype, hidden, rows, mixed):
    import torch
    w = _levels(rows, hidden, dtype, mixed)
    prev = F.fold_level_launches(True)
    try:
        for on in (True, False):
            F.fold_level_launches(on)
            dev, saved = _sizes(w)
            assert dev.fwd_bytes > (saved + 255) // 256 * 256  # the high levels do split
            guard = 64 << 20
            ws = torch.full((dev.fwd_bytes + guard,), 0xA5, dtype=torch.uint8, device="cuda")
            dev.ws = ws[:dev.fwd_bytes]
            dev.forward()
            torch.cuda.synchronize()
            assert bool((ws[dev.fwd_bytes:] == 0xA5).all()), on
    finally:
        F.fold_level_launches(prev)
