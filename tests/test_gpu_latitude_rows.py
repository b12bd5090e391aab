"""Batches and server slots whose queries have their own row of the latitude
table against the plain path, which reads the table itself: below, at and above
the speed ratios that the table covers, in one batch with queries without a row
(S = 0, S outside the table, a box control volume), at the particle count from
which rows are made, and in a workspace without room for them.  Bit for bit."""
import ctypes

import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu

N = 1 << 17  # eight queries: 2^20 particles, the least that makes rows
SPEEDS = (0.0, 0.2, 0.25, 1.0, 4.0, 10.0, 10.5, 2.0)


@pytest.fixture(scope="module")
def T():
    from paper_1312_3691_amd import tpmc
    return tpmc


@pytest.fixture(scope="module")
def ctx(T):
    return T.Context(0)


def _queries(n=N):
    return [I.query(q=tuple(qq), S=S, alpha=0.8, n=n, seed=60 + i, cv_box=S == 2.0)
            for i, (S, qq) in enumerate(zip(SPEEDS, I.random_quats(len(SPEEDS), 4)))]


def _same(T, plain, got, what):
    for i, (p, g) in enumerate(zip(plain, got)):
        for k in T.same_on_every_path(p):
            assert np.array_equal(np.asarray(p[k]), np.asarray(g[k]), equal_nan=True), (what, i, k)


@pytest.mark.parametrize("make", [I.plate, I.capped_cylinder, lambda: I.satellite(2000)],
                         ids=["plate", "cylinder", "satellite"])
@pytest.mark.parametrize("n", [N - 1, N, N + 1])
def test_rows_equal_the_table(ctx, T, make, n):
    mesh = ctx.build_mesh(*make())
    qs = _queries(n)
    plain, pr = T.run(mesh, qs, A_ref=1.0)
    pr.close()
    b = T.Batch(mesh, qs)
    for _ in range(2):
        _same(T, plain, b.launch(use_graph=True).results(A_ref=1.0), n)
    b.close()
    arr = T._queries(qs)
    nbytes = ctypes.c_uint64()
    T._check(T._lib.tpmc_batch_workspace_bytes(ctx._h, mesh._h, arr, len(qs), ctypes.byref(nbytes)))
    buf, ptr, _ = T._workspace(nbytes.value, ctx.device)
    h = ctypes.c_void_p()
    T._check(T._lib.tpmc_batch_create(ctx._h, mesh._h, arr, len(qs), ctypes.c_void_p(ptr), nbytes.value - 256,
                                      ctypes.byref(h)))
    T._check(T._lib.tpmc_batch_launch(ctx._h, h, 0))
    res = (T.Result * len(qs))()
    T._check(T._lib.tpmc_batch_results(ctx._h, h, (ctypes.c_double * 3)(), 1.0, res))
    _same(T, plain, [T.result_dict(r) for r in res], "no room")
    T._lib.tpmc_destroy_batch(h)
    del buf
    mesh.close()


@pytest.mark.parametrize("n", [32_767, 32_768, 70_001])  # rows from 32768 particles a slot
def test_slots_equal_the_table(ctx, T, n):
    mesh = ctx.build_mesh(*I.capped_cylinder())
    qs = _queries(n)
    plain, pr = T.run(mesh, qs, A_ref=1.0)
    pr.close()
    words = 7 * mesh.nt
    srv = T.Server(ctx, len(qs), words * len(qs))
    for turn in range(2):  # the second turn reuses each slot's row for another query
        order = list(range(len(qs)))[::-1 if turn else 1]
        tiles = srv.admit_many([(slot, mesh, qs[i], words * slot) for slot, i in enumerate(order)])
        srv.step([(slot, 0, t) for slot, t in enumerate(tiles)])
        got = srv.collected(srv.collect(range(len(qs))))
        _same(T, [plain[i] for i in order], got, (n, turn))
    srv.close()
    mesh.close()
