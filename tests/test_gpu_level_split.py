"""fp32 levels whose K is cut by rounds of tiles, against the oracle, forward and backward: around the smallest level
that the rule takes (96 tiles), one row tile past a full round, and levels of several cells side by side."""
import pytest

from tests import gpu_common as C
from tests.test_gpu_narrow import _levels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,rows,mixed", [
    (256, 1408, False), (256, 1409, False), (512, 2050, False), (512, 641, False), (500, 1100, False),
    (256, 2200, True),
])
def test_level_split(hidden, rows, mixed):
    w = _levels(rows, hidden, "f32", mixed)
    errs = C.compare_all(w, C.run_device(w), C.run_oracle(w))
    print(hidden, rows, mixed, errs)


@pytest.mark.parametrize("hidden,rows", [(320, 1243), (370, 1115), (640, 731)])
def test_level_split_of_widths_between_xcd_shares(hidden, rows):
    """Widths whose columns do not divide by the eight XCDs: the slices are counted by the fullest one."""
    w = _levels(rows, hidden, "f32", False)
    errs = C.compare_all(w, C.run_device(w), C.run_oracle(w))
    print(hidden, rows, errs)
