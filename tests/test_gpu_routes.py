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


KIND_ID = {"fp64": 0, "fp32": 1, "bf16": 2, "fp32w": 3, "bf16w": 3}
KIND_KEY = ("fp64", "fp32", "bf16", "fp32w")


def instances():
    """Kind, directions and shape of every instance of the tiled kernel."""
    for kind in KINDS:
        for D in range(4):
            if kind in ("fp64", "fp32w", "bf16w") and D >= 2:
                yield kind, D, "4x4"
                continue
            yield kind, D, "8x8"
            if D in (1, 3):
                yield kind, D, "4x8"
            if D == 1 and kind != "bf16":
                yield kind, D, "8x4"


def forced(tmp_path, kind, D, b, shape):
    """Options that set `shape` for the kind and 8x8 or 4x4 for the others."""
    path = tmp_path / f"shapes_{kind}_{D}_{shape}"
    lines = []
    for k in KIND_KEY:
        wide = k in ("fp64", "fp32w") and D >= 2
        sh = shape if k == KIND_KEY[KIND_ID[kind]] else ("4x4" if wide else "8x8")
        lines.append(json.dumps({"key": f"gfx950/{k}/D{D}/k{(b + 3) // 4}/s1", "shape": sh, "ms": {}}))
    path.write_text("\n".join(lines) + "\n")
    return dict(skip="bound", tune=True, tune_cache=str(path), **KINDS[kind])


@pytest.mark.parametrize("b", [13, 9, 16])
@pytest.mark.parametrize("kind,D,shape", list(instances()))
def test_whole_subtiles_of_every_instance(knob, tmp_path, kind, D, shape, b):
    # small systems run in parts, the same for every shape; larger ones take the
    # instance of the shape, here forced: all results are those of the parts.
    # The sums over a sub-tile's outputs follow its shape.
    s = W.batch_systems(sizes=[29], n_dir=D, b=b)[0]
    parts = T.solve(s, **dict(KINDS[kind], skip="bound"))[0]
    knob("TC2_TEST_FINE_SUBS", 0)
    whole = T.solve(s, **forced(tmp_path, kind, D, b, shape))[0]
    assert whole.tile_shape[KIND_ID[kind]] == ("8x8", "4x8", "8x4", "4x4").index(shape)
    assert whole.ms_tune == 0.0
    for x, y in zip([parts.X0] + parts.X1, [whole.X0] + whole.X1):
        assert np.array_equal(x.row_ptr, y.row_ptr) and np.array_equal(x.col, y.col)
        assert np.array_equal(x.val, y.val)
    assert parts.branches == whole.branches and parts.iters == whole.iters
    assert parts.executed_flops == whole.executed_flops
    assert parts.screened_blocks == whole.screened_blocks
    assert whole.alpha == pytest.approx(parts.alpha, rel=1e-12)
    # panel passes of 8 columns, and every product issued: equal matrices again
    for name, value in (("TC2_TEST_KL_CHUNK", 8), ("TC2_TEST_NO_ZERO_SKIP", 1)):
        knob(name, value)
        other = T.solve(s, **forced(tmp_path, kind, D, b, shape))[0]
        for x, y in zip([other.X0] + other.X1, [whole.X0] + whole.X1):
            assert np.array_equal(x.row_ptr, y.row_ptr) and np.array_equal(x.col, y.col)
            assert np.array_equal(x.val, y.val)


@pytest.mark.parametrize("kind,D", [("fp64", 0), ("fp64", 1), ("fp64", 2), ("fp64", 3), ("fp32w", 1),
                                    ("fp32w", 3), ("bf16w", 2)])
def test_trace_groups_of_whole_subtiles(knob, kind, D):
    # the traces of a whole sub-tile are summed in the groups that the parts
    # use, or (waves per column 1) by column of the sub-tile
    s = W.batch_systems(sizes=[61], n_dir=D, b=13)[0]
    a = T.solve(s, **KINDS[kind])[0]
    knob("TC2_TEST_FINE_SUBS", 0)
    b = T.solve(s, **KINDS[kind])[0]
    same(a, b)
    knob("TC2_TEST_WAVES_PER_COLUMN", 1)
    c = T.solve(s, **KINDS[kind])[0]
    assert c.alpha == pytest.approx(b.alpha, rel=1e-12)
    for x, y in zip([c.X0] + c.X1, [b.X0] + b.X1):
        assert np.array_equal(x.val, y.val)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("kind", ["fp32", "bf16", "fp32w", "bf16w"])
def test_reduced_solve_that_ends_in_its_leading_fp64_updates(kind, graph):
    # the closing pair then starts from an FP64 iterate: two more FP64 updates of
    # the converged X0, and systems without or with all states occupied unchanged
    opts = dict(KINDS[kind], fp64_first=60, skip="bound", graph=graph)
    s = W.batch_systems(sizes=[29, 12, 17], n_dir=2, b=6)
    s[1].n_occ, s[2].n_occ = 0, s[2].H.n
    ref = T.solve(s, skip="bound")
    for trivial in (False, True):
        got = T.solve(s[1:] if trivial else s, **opts)
        for a, b in zip(got, ref[1:] if trivial else ref):
            assert a.status_name == b.status_name
            for x, y in zip([a.X0] + a.X1, [b.X0] + b.X1):
                if a is got[0] and not trivial:
                    d = np.abs(dense(x) - dense(y)).max()
                    assert d < 1e-5, d  # ten times the drop threshold
                else:
                    assert np.array_equal(x.row_ptr, y.row_ptr) and np.array_equal(x.col, y.col)
                    assert np.array_equal(x.val, y.val)


def dense(m):
    A = np.zeros((m.nb, m.nb, m.b, m.b))
    A[np.repeat(np.arange(m.nb), np.diff(m.row_ptr)), m.col] = m.val
    return A


@pytest.mark.parametrize("opts", [dict(), dict(FP32, fp64_first=2)])
def test_advance_of_systems_without_an_update(opts):
    # no state, or every state, occupied: a solve has no update to run, and a call
    # returns after one such solve
    s = W.batch_systems(sizes=[9, 17], n_dir=1, b=5)
    s[0].n_occ, s[1].n_occ = 0, s[1].H.n
    ref = T.solve(s, **opts)
    sv = T.Solver(s, **opts)
    for _ in range(2):
        p, r = sv.advance(5)
        assert p["updates"] == 0 and p["solves_completed"] == 1 and not p["solve_open"]
        for a, b in zip(r, ref):
            same(a, b)
    sv.close()
