"""Memory and waits of schedules: fold_trim gives everything idle back, a freed schedule has waited for work on every
stream, and a schedule can be made (not only freed) while another thread records a stream."""
import threading

import numpy as np
import pytest

from paper_1702_02181_amd import fold as F
from paper_1702_02181_amd import gen
from tests import gpu_common as C

pytestmark = pytest.mark.gpu


def _make(w):
    import torch
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    return F.Schedule(i32(w.graph_ptr), i32(w.node_op), i32(w.child_ptr), i32(w.child_idx), i32(w.node_input),
                      [(o.kind, o.arity, o.has_input, o.param_set) for o in w.ops], w.leaf_table.shape[0])


def _free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_trim_gives_idle_memory_back():
    import torch
    w = gen.config2(num_graphs=1200, leaves=128, hidden=2)  # 306,000 nodes: blocks of some 40 and 50 MB
    F.fold_trim()  # earlier schedules' blocks: those of less than 2 MB share allocations of the GPU driver and do not show as free
    keep = _make(w)
    other = _make(w)
    want = C.oracle_schedule(w)
    del other
    torch.cuda.empty_cache()
    before = _free_bytes()
    freed = F.fold_trim()
    assert freed >= 4 * 23 * w.num_nodes  # the freed schedule's arrays at least (23 ints a node and more)
    assert _free_bytes() - before >= freed
    assert F.fold_trim() == 0
    C.assert_schedule_equal(keep.arrays(), want)  # the one alive is whole, and new ones are made
    C.assert_schedule_equal(_make(w).arrays(), want)


def test_free_waits_for_every_stream():
    """A schedule freed while a forward that reads it is queued on another stream: the wait covers that stream, so the
    block is not handed on under the forward."""
    import torch
    from paper_1702_02181_amd.runner import DeviceRun
    w = gen.config2(num_graphs=64, leaves=64, hidden=256)
    dev = DeviceRun(w)
    dev.forward()
    torch.cuda.synchronize()
    want = dev.h_pool.clone()
    other = gen.config2(num_graphs=64, leaves=64, hidden=256, seed=9)
    st = torch.cuda.Stream()
    dev.h_pool.zero_()
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(st):
        for _ in range(50):
            dev.forward()
        done.record()
    F.fold_sched_free(dev.sched.handle)
    assert done.query()
    dev.sched.handle = None
    C.assert_schedule_equal(_make(other).arrays(), C.oracle_schedule(other))
    torch.cuda.synchronize()
    assert torch.equal(dev.h_pool, want)


@pytest.mark.parametrize("graphs", [4, 400])  # the one-launch schedule and the tiled one
@pytest.mark.parametrize("mode", ["thread_local", "relaxed"])
def test_schedule_made_while_another_thread_captures(mode, graphs):
    import torch
    w = gen.config2(num_graphs=graphs, leaves=24, hidden=2)
    _make(w)  # torch's own blocks for the batch are there
    x, y = torch.arange(64, dtype=torch.float32, device="cuda"), torch.zeros(64, device="cuda")
    st = torch.cuda.Stream()
    got = []

    def make(arrays):
        try:
            with torch.cuda.stream(st):
                got.append(F.Schedule(*arrays, [(o.kind, o.arity, o.has_input, o.param_set) for o in w.ops],
                                      w.leaf_table.shape[0]))
        except BaseException as e:  # noqa: BLE001 -- reported by the main thread
            got.append(e)

    arrays = [torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
              for a in (w.graph_ptr, w.node_op, w.child_ptr, w.child_idx, w.node_input)]
    torch.cuda.synchronize()
    for trim in (False, True):  # with blocks at hand, and with new ones
        if trim:
            F.fold_trim()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, capture_error_mode=mode):
            torch.mul(x, 2, out=y)
            t = threading.Thread(target=make, args=(arrays,))
            t.start()
            t.join()
        for k in range(3):
            y.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, 2 * x), k
        assert isinstance(got[-1], F.Schedule), got
        C.assert_schedule_equal(got.pop().arrays(), C.oracle_schedule(w))
