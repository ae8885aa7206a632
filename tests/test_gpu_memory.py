"""Device buffers kept for reuse: solves of several threads at once, with
released buffers passing between them, equal the same solves one by one."""
import threading
import time

import numpy as np
import pytest
import torch

from paper_2009_03551_amd import tc2 as T
from paper_2009_03551_amd import workloads as W

pytestmark = pytest.mark.gpu


def matrices(r):
    return [a for m in [r.X0] + r.X1 for a in (m.row_ptr, m.col, m.val)]


@pytest.mark.parametrize("variant", [dict(), dict(precision="fp32", wide=True, fp64_first=2, closing_fp64=2)])
def test_threads_share_released_buffers(variant):
    systems = [W.config_system("chain64", n=29 + 8 * k, b=5 + k, occ=2, eps=1e-6, seed=k) for k in range(4)]
    alone = [matrices(T.solve(s, **variant)[0]) for s in systems]
    out = [[] for _ in systems]

    def work(k):
        for _ in range(5):
            out[k].append(matrices(T.solve(systems[k], **variant)[0]))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(systems))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    T.trim_memory(0)  # the kept buffers go back; the next solve starts from none
    for k, s in enumerate(systems):
        out[k].append(matrices(T.solve(s, **variant)[0]))
        assert len(out[k]) == 6
        for got in out[k]:
            assert all(np.array_equal(a, b) for a, b in zip(got, alone[k]))


@pytest.mark.parametrize("graph", [False, True])
def test_threads_release_large_buffers(graph):
    """Value buffers of several mapped chunks of 256 MB (343 atoms in three
    directions), released by one thread while another one grows its own."""
    systems = [W.config_system("cube20", L=7, seed=3 + k) for k in range(2)]
    opts = dict(skip="bound", graph=graph)
    alone = [matrices(T.solve(s, **opts)[0]) for s in systems]
    # stored blocks (16 x 16 FP64 values of four matrices) of the iterate
    assert all(m[1].size * 4 * 2048 > 256 << 20 for m in alone)
    same = [[] for _ in systems]

    def work(k):
        for _ in range(3):
            got = matrices(T.solve(systems[k], **opts)[0])
            same[k].append(all(np.array_equal(a, b) for a, b in zip(got, alone[k])))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(systems))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert same == [[True] * 3] * 2


@pytest.mark.parametrize("what", ["solve", "mlp", "lowdin", "wait"])
def test_captures_beside_other_calls(what):
    """Solves that capture their updates while another thread sets up, solves and
    frees systems, calls the skip network or orthogonalises, or waits for the
    whole device (which ends a capture: it is taken again)."""
    s = W.config_system("chain64", n=61, b=5, occ=2, eps=1e-6, seed=4)
    small = W.config_system("chain64", n=29, b=5, occ=2, eps=1e-6, seed=5)
    S = W.make_overlap(small, amp=0.1, seed=6)
    rng = np.random.default_rng(7)
    theta = rng.normal(0.0, 0.3, T.MLP_PARAMS).astype(np.float32)
    x = rng.normal(0.0, 0.5, (500, T.MLP_IN)).astype(np.float32)
    y = (rng.random(500) < 0.2).astype(np.float32)
    calls = {"solve": lambda: matrices(T.solve(small)[0]),
             "mlp": lambda: [T.mlp_grad(theta, x, y)[0], T.mlp_forward(theta, x)],
             "lowdin": lambda: [T.lowdin(S, small.H, small.H1, eps=1e-8).Z.val]}
    opts = dict(skip="bound", graph=True)
    alone = matrices(T.solve(s, **opts)[0])
    if what in calls:
        other = calls[what]()
    stop = threading.Event()
    waits = [0]
    failed = []

    def beside():
        while not stop.is_set():
            try:
                if what == "wait":
                    try:
                        torch.cuda.synchronize()
                    except RuntimeError:  # refused during a capture, which it ends
                        pass
                    waits[0] += 1
                    time.sleep(0.002)
                else:
                    got = calls[what]()
                    if not all(np.array_equal(a, b) for a, b in zip(got, other)):
                        failed.append("other results")
            except Exception as e:
                failed.append(repr(e))

    t = threading.Thread(target=beside)
    t.start()
    try:
        for _ in range(25):
            got = matrices(T.solve(s, **opts)[0])  # a new context: captures anew
            assert all(np.array_equal(a, b) for a, b in zip(got, alone))
    finally:
        stop.set()
        t.join()
    assert not failed, failed[:3]
