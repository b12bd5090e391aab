"""The SAH build's three stages (big nodes in chunks, one workgroup per node, one
wave per subtree) at the sizes where they meet, on shuffled soups, a convex
body and coincident triangles: results, per-triangle loads and first hits equal
those on the LBVH bit for bit."""
import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_1312_3691_amd import tpmc
    return tpmc


@pytest.fixture(scope="module")
def ctx(T):
    return T.Context(0)


def _soup(n, seed, clustered):
    """n small triangles; clustered: centres cubed towards the origin, so that splits are uneven."""
    r = np.random.default_rng(seed)
    c = r.uniform(-1, 1, (n, 1, 3))
    V = ((c ** 3 if clustered else c) + r.normal(0, 0.02, (n, 3, 3))).reshape(-1, 3).astype(np.float32)
    return V, np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)


def _same(n, distinct):
    """n copies of `distinct` triangles (no plane separates the copies)."""
    V, Tr = _soup(distinct, 5, False)
    return V, np.tile(Tr, (n // distinct + 1, 1))[:n]


BODIES = ([("soup%d" % n, _soup(n, n, n % 2 == 0)) for n in (2, 3, 31, 32, 33, 64, 65, 1023, 1024, 1025, 1026, 5000, 30_001)]
          + [("same%d" % n, _same(n, d)) for n, d in ((40, 1), (1500, 2), (3000, 3))]
          + [("sphere", I.icosphere(4)), ("satellite", I.satellite(20_000))])


@pytest.mark.parametrize("name,body", BODIES, ids=[b[0] for b in BODIES])
def test_sah_equals_lbvh(ctx, T, name, body):
    V, Tr = body
    q = I.query(S=3.0, n=20_001, seed=8, alpha=0.9, q=tuple(I.random_quats(1, 4)[0]))
    got = {}
    for builder in ("sah", "lbvh"):
        mesh = ctx.build_mesh(V, Tr, builder=builder)
        assert 1 <= mesh.info["depth"] <= 64
        res, pr = T.run(mesh, [q], A_ref=1.0, first_tri=True)
        got[builder] = (res[0], pr.tally(), pr.first_tri.cpu().numpy())
        pr.close()
        mesh.close()
    a, b = got["sah"], got["lbvh"]
    assert a[0]["guard_trips"] == 0 and b[0]["guard_trips"] == 0
    for k in T.same_on_every_path(a[0]):
        assert np.array_equal(np.asarray(a[0][k]), np.asarray(b[0][k])), (name, k)
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
