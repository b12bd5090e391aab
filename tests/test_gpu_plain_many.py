"""Plain runs of several queries in one launch, at the sizes where a wave's share
of particles and the workgroups of a query change, and with both tally kinds
mixed: seeded states, first triangles, per-triangle loads and results equal
those of a run of each query alone, and its results those of a batch, bit for
bit."""
import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu

MESHES = {"plate": I.plate, "cylinder": I.capped_cylinder, "sphere": lambda: I.icosphere(3),
          "satellite": lambda: I.satellite(2000)}


def _outputs(pr, n):
    states = [p.cpu().numpy() for p in pr.planes()]
    return states, pr.first_tri.cpu().numpy()


@pytest.mark.parametrize("kind", sorted(MESHES))
@pytest.mark.parametrize("sizes", [(1, 64, 65, 255, 256, 257), (262_143, 1, 262_145), (3, 700_001, 2000, 262_144)],
                         ids=lambda s: "x".join(map(str, s[:3])))
def test_many_equal_each_alone(kind, sizes):
    from paper_1312_3691_amd import tpmc
    ctx = tpmc.Context(0)
    mesh = ctx.build_mesh(*MESHES[kind]())
    qs = [I.query(q=tuple(qq), S=3.0 + i, alpha=0.9, n=n, seed=80 + i, flags=i % 2)  # every other: totals only
          for i, (n, qq) in enumerate(zip(sizes, I.random_quats(len(sizes), 6)))]
    many, pr = tpmc.run(mesh, qs, A_ref=1.0, first_tri=True)
    again = pr.forces(A_ref=1.0)  # the totals are cleared and summed again
    states, first = _outputs(pr, len(qs))
    off = 0
    for i, q in enumerate(qs):
        alone, one = tpmc.run(mesh, [q], A_ref=1.0, first_tri=True)
        s1, f1 = _outputs(one, 1)
        n = q["n"]
        for k in range(6):
            assert np.array_equal(states[k][off:off + n], s1[k]), (i, k)
        assert np.array_equal(first[off:off + n], f1), i
        assert (f1 >= -1).all()  # every particle was followed
        if not q["flags"]:
            assert np.array_equal(pr.tally(i), one.tally(0)), i
        b = tpmc.Batch(mesh, [q])
        batch = b.launch().results(A_ref=1.0)[0]
        b.close()
        assert many[i]["rays"] == n
        for k in tpmc.same_on_every_path(many[i]):
            for other in (alone[0], batch, again[i]):
                assert np.array_equal(np.asarray(many[i][k]), np.asarray(other[k]), equal_nan=True), (i, k)
        one.close()
        off += n
    pr.close()
    mesh.close()
