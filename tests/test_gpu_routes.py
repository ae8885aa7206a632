"""Routes that an update takes by the size of a problem, against each other on
the same problem: the environment moves the limits between them."""
import json

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


def tuned(path, s, **kw):
    r = T.solve(s, skip="bound", tune=True, tune_cache=str(path), **kw)[0]
    return r, [json.loads(x) for x in path.read_text().splitlines()]


def test_a_small_problem_is_tuned_by_whole_subtiles(tmp_path):
    # 64 atoms run in parts of sub-tiles, the same for every shape; an 8 x 8
    # sub-tile by one workgroup takes 1.8 times as long as its halves by two
    # (0.20 ms against 0.11)
    s = W.config_system("chain64")
    ms = [tuned(tmp_path / f"t{k}", s)[1][0]["ms"] for k in range(3)]
    assert min(m["8x8"] for m in ms) > 1.2 * max(m["8x4"] for m in ms), ms


def test_a_shape_tuned_on_a_small_problem_stays_there(tmp_path):
    small, large = W.config_system("cube10", L=4), W.config_system("cube10", L=8)
    path = tmp_path / "tune"
    a, lines = tuned(path, small)
    assert len(lines) == 1 and lines[0]["parts"] == 1 and a.ms_tune > 0.0
    b, lines = tuned(path, large, export=False)
    assert len(lines) == 2 and lines[1]["parts"] == 0 and b.ms_tune > 0.0
    c, lines = tuned(path, large, export=False)
    assert len(lines) == 2 and c.ms_tune == 0.0 and c.tile_shape == b.tile_shape
    d, lines = tuned(path, small)
    assert len(lines) == 2 and d.ms_tune == 0.0


def test_shapes_timed_with_another_kernel_are_timed_again(tmp_path):
    s = W.config_system("cube10", L=4)
    path = tmp_path / "tune"
    path.write_text('{"key": "gfx950/fp64/D1/k4/s1", "shape": "8x4", '
                    '"ms": {"8x8": 0.2, "4x8": 0.2, "8x4": 0.1}}\n')
    a, lines = tuned(path, s)
    assert a.ms_tune > 0.0 and len(lines) == 2
    b, lines = tuned(path, s)
    assert b.ms_tune == 0.0 and len(lines) == 2 and b.tile_shape == a.tile_shape


FP32 = dict(precision="fp32", closing_fp64=2)
KINDS = {"fp64": dict(), "fp32": FP32, "bf16": dict(precision="bf16", closing_fp64=2),
         "fp32w": dict(FP32, wide=True, fp64_first=2),
         "bf16w": dict(precision="bf16", wide=True, fp64_first=2, closing_fp64=2)}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("D", [0, 1, 2, 3])
def test_learned_screen_in_parts_equals_whole_subtiles(knob, kind, D):
    # the same features, logits and decisions, whichever workgroup computes an
    # output: equal matrices and logs (samples in any order).  45 atoms: six
    # clusters, the last one ragged
    s = W.batch_systems(sizes=[45], n_dir=D, b=13 if D != 2 else 6)[0]
    theta = np.zeros(T.MLP_PARAMS, dtype=np.float32)
    theta[:] = np.random.default_rng(2).normal(0.0, 0.3, T.MLP_PARAMS)

    def run():
        a = T.solve(s, skip="mlp", mlp_weights=theta, mlp_threshold=0.5, mlp_bound_cap=2.0,
                    **KINDS[kind])[0]
        sv = T.Solver(s, skip="bound", log_capacity=200000, **KINDS[kind])
        b = sv.run()[0]
        x, y = sv.log()
        sv.close()
        order = np.lexsort(np.concatenate([x.T, y[None]]))
        return a, b, x[order], y[order]

    a0, b0, x0, y0 = run()
    knob("TC2_TEST_FINE_SUBS", 0)
    a1, b1, x1, y1 = run()
    same(a0, a1)
    same(b0, b1)
    assert a0.mlp_skipped_blocks == a1.mlp_skipped_blocks
    assert a0.screened_blocks == a1.screened_blocks and b0.screened_blocks == b1.screened_blocks
    assert len(y0) > 0 and np.array_equal(x0, x1) and np.array_equal(y0, y1)
