"""Batched launches at the sizes where the cut into units changes: fewer
particles than a batch, than one batch per wave, just above, uneven queries in
one launch, many small queries (whose last units only the waves that started
on them take), and a workspace without room for the copies of the scalar sums.
Every result equals the plain path's bit for bit."""
import ctypes

import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu

MESHES = {"plate": I.plate, "cylinder": I.capped_cylinder, "sphere": lambda: I.icosphere(3),
          "satellite": lambda: I.satellite(2000)}


@pytest.fixture(scope="module")
def T():
    from paper_1312_3691_amd import tpmc
    return tpmc


@pytest.fixture(scope="module")
def ctx(T):
    return T.Context(0)


def _same(T, plain, got, what):
    for i, (p, g) in enumerate(zip(plain, got)):
        for k in T.same_on_every_path(p):
            assert np.array_equal(np.asarray(p[k]), np.asarray(g[k]), equal_nan=True), (what, i, k)


@pytest.mark.parametrize("kind", sorted(MESHES))
@pytest.mark.parametrize("totals", [False, True])
@pytest.mark.parametrize("sizes", [(1,), (63, 64, 65), (1000, 1, 130_000), (262_143,), (262_209, 5), (700_001,),
                                   tuple(16_200 + i for i in range(150))], ids=lambda s: "x".join(map(str, s[:4])))
def test_batch_equals_plain_at_unit_edges(ctx, T, kind, totals, sizes):
    mesh = ctx.build_mesh(*MESHES[kind]())
    qs = [I.query(q=tuple(qq), S=3.0 + i % 7, alpha=0.9, n=n, seed=40 + i, flags=1 if totals else 0)
          for i, (n, qq) in enumerate(zip(sizes, I.random_quats(len(sizes), 3)))]
    plain, pr = T.run(mesh, qs, A_ref=1.0)
    pr.close()
    b = T.Batch(mesh, qs)
    for _ in range(2):
        got = b.launch(use_graph=True).results(A_ref=1.0)
        assert [g["rays"] for g in got] == list(sizes)
        _same(T, plain, got, (kind, totals, sizes))
    b.close()
    mesh.close()


def test_batch_without_room_for_copies(ctx, T):
    mesh = ctx.build_mesh(*I.capped_cylinder())
    qs = [I.query(S=4.0, n=300_001, seed=9), I.query(S=2.0, n=40_000, seed=10)]
    plain, pr = T.run(mesh, qs, A_ref=1.0)
    pr.close()
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
    _same(T, plain, [T.result_dict(r) for r in res], "no copies")
    T._lib.tpmc_destroy_batch(h)
    del buf
    mesh.close()
