"""Routes that an update takes by the size of a problem, against each other on
the same problem: the environment moves the limits between them."""
import numpy as np
import pytest

from paper_2009_03551_amd import tc2 as T
from paper_2009_03551_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture
def knob(monkeypatch):
    """Sets a limit, read when a context is made."""
    return lambda name, value: monkeypatch.setenv(name, str(value))


def same(a, b):
    assert a.branches == b.branches and a.iters == b.iters and a.alpha == b.alpha
    for x, y in zip([a.X0] + a.X1, [b.X0] + b.X1):
        assert np.array_equal(x.row_ptr, y.row_ptr) and np.array_equal(x.col, y.col)
        assert np.array_equal(x.val, y.val)


@pytest.mark.parametrize("sizes,bound", [((61,), 0), ((9, 1, 40), 0), ((61,), 20000)])
def test_panel_columns_counted_or_bounded(knob, sizes, bound):
    # the panel buffers are sized by the stored blocks, or, where those are many,
    # by the columns read back (20000: some updates of the solve each way); the
    # systems of a batch stop at different updates
    s = [W.config_system("chain64", n=n, b=5, occ=2, eps=1e-6, seed=3 + n) for n in sizes]
    a = T.solve(s)
    knob("TC2_TEST_PANEL_BOUND", bound)
    b = T.solve(s)
    for x, y in zip(a, b):
        same(x, y)
