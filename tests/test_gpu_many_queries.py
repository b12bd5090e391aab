"""Batches of more queries than the launch has workgroups (a workgroup then works
off several queries of its own): equal, tiny and very uneven queries, each tally
kind.  Every result equals the plain path's bit for bit, over repeated launches."""
import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu

MESHES = {"plate": I.plate, "cylinder": I.capped_cylinder, "satellite": lambda: I.satellite(1000)}
SIZES = {"1025x64": [64] * 1025, "2500x1": [1] * 2500, "3000x130": [130] * 3000,
         "log": [int(v) for v in np.exp(np.random.default_rng(1).uniform(0.0, np.log(30_000.0), 1400))],
         "one large": [100] * 1100 + [1_000_000] + [300] * 200}


@pytest.fixture(scope="module")
def T():
    from paper_1312_3691_amd import tpmc
    return tpmc


@pytest.fixture(scope="module")
def ctx(T):
    return T.Context(0)


@pytest.mark.parametrize("kind", sorted(MESHES))
@pytest.mark.parametrize("totals", [False, True])
@pytest.mark.parametrize("sizes", sorted(SIZES))
def test_batch_equals_plain(ctx, T, kind, totals, sizes):
    mesh = ctx.build_mesh(*MESHES[kind]())
    n = SIZES[sizes]
    qs = [I.query(q=tuple(qq), S=2.0 + i % 9, alpha=0.9, n=k, seed=40 + i, flags=1 if totals else 0)
          for i, (k, qq) in enumerate(zip(n, I.random_quats(len(n), 3)))]
    plain, pr = T.run(mesh, qs, A_ref=1.0)
    pr.close()
    b = T.Batch(mesh, qs)
    for _ in range(2):
        got = b.launch(use_graph=True).results(A_ref=1.0)
        assert [g["rays"] for g in got] == n
        for i, (p, g) in enumerate(zip(plain, got)):
            for k in T.same_on_every_path(p):
                assert np.array_equal(np.asarray(p[k]), np.asarray(g[k]), equal_nan=True), (kind, totals, sizes, i, k)
    b.close()
    mesh.close()


def test_more_queries_than_one_launch_of_a_stage_takes(ctx, T):
    """70001 queries: the plain path's stages and the finalisation run in chunks."""
    mesh = ctx.build_mesh(*I.plate())
    qs = [I.query(S=2.0 + i % 9, alpha=0.9, n=1 + i % 3, seed=i) for i in range(70_001)]
    plain, pr = T.run(mesh, qs, A_ref=1.0)
    pr.close()
    b = T.Batch(mesh, qs)
    got = b.launch().results(A_ref=1.0)
    assert len(got) == len(plain) == len(qs)
    for i, (q, p, g) in enumerate(zip(qs, plain, got)):
        assert p["rays"] == g["rays"] == q["n"], i
        for k in ("CD", "hits", "missed", "segments", "escaped", "Qhat"):
            assert p[k] == g[k], (i, k)
        assert (p["F_over_q"] == g["F_over_q"]).all(), i
    b.close()
    mesh.close()
