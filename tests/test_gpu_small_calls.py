"""Queries passed in a launch's arguments or by copy, results written to pinned
host memory or copied, per-triangle sums added up by the finalisation or by a
reduction of their own: each on both sides of its limit, every result equal bit
for bit (the same counters, exact sums) to that of totals kept in registers."""
import threading

import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu


def _equal(T, a, b, what):
    assert len(a) == len(b)
    for i, (x, y) in enumerate(zip(a, b)):
        for k in T.same_on_every_path(x):
            assert np.array_equal(np.asarray(x[k]), np.asarray(y[k]), equal_nan=True), (what, i, k)


@pytest.mark.parametrize("body", ["plate", 2044, 2048, 2052])
@pytest.mark.parametrize("nq", [1, 4, 5, 64, 65])
def test_small_calls(body, nq):
    from paper_1312_3691_amd import tpmc as T
    ctx = T.Context(0)
    mesh = ctx.build_mesh(*(I.plate() if body == "plate" else I.capped_cylinder(segments=body // 4)))
    assert body == "plate" or mesh.nt == body
    qs = [I.query(q=tuple(qq), S=2.0 + i % 5, alpha=0.9, n=500 + i, seed=90 + i)
          for i, qq in enumerate(I.random_quats(nq, 8))]
    want, pr = T.run(mesh, [dict(q, flags=T.Q_NO_TRIANGLE_TALLY) for q in qs], x_ref=(0.1, 0.2, 0.3), A_ref=2.0)
    pr.close()
    plain, pr = T.run(mesh, qs, x_ref=(0.1, 0.2, 0.3), A_ref=2.0)
    _equal(T, want, plain, "plain")
    _equal(T, want, pr.forces((0.1, 0.2, 0.3), 2.0), "forces again")
    pr.close()
    b = T.Batch(mesh, qs)
    for graph in (False, True, True):
        b.launch(use_graph=graph)
        for _ in range(2):
            _equal(T, want, b.results((0.1, 0.2, 0.3), 2.0), ("batch", graph))
    b.close()
    for _ in range(2):
        _equal(T, want, T.batch_run_noalloc(mesh, qs, (0.1, 0.2, 0.3), 2.0), "noalloc")
    mesh.close()


def test_results_from_several_threads():
    from paper_1312_3691_amd import tpmc as T
    ctx = T.Context(0)
    mesh = ctx.build_mesh(*I.capped_cylinder())
    runs = []
    for k in range(4):
        b = T.Batch(mesh, [I.query(S=3.0 + k, n=3000, seed=k)])
        runs.append((b, b.launch().results()))
    wrong = []

    def work(b, want):
        for _ in range(50):
            got = b.results()
            for k in T.same_on_every_path(want[0]):
                if not np.array_equal(np.asarray(got[0][k]), np.asarray(want[0][k]), equal_nan=True):
                    wrong.append(k)

    threads = [threading.Thread(target=work, args=r) for r in runs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    for b, _ in runs:
        b.close()
    mesh.close()


def test_more_contexts_than_pinned_blocks():
    from paper_1312_3691_amd import tpmc as T
    for _ in range(2):  # blocks are given back
        ctxs = [T.Context(0) for _ in range(34)]
        got = []
        for c in ctxs:
            mesh = c.build_mesh(*I.plate())
            got.append(T.batch_run_noalloc(mesh, [I.query(S=4.0, n=2000, seed=3)]))
            mesh.close()
        for g in got[1:]:
            _equal(T, got[0], g, "contexts")
        for c in ctxs:
            c.close()
