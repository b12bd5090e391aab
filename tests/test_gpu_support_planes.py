"""Supporting planes of a build at the vertex counts where it changes from one pass
over all vertices to a spread sample and a second pass: a flat grid with one small
roof above it, the roof's vertices first, last or in the middle of the list.  The
grid's plane is a supporting one but for the roof: a pass that misses its vertices
would end the grid's re-emissions there.  Counts against the oracle: equal seeds, so
they differ only where FP32 moves a grazing ray, a thousandth of the hits at most (as
in the workloads' parity)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1312_3691_amd import inputs as I

pytestmark = pytest.mark.gpu


def _grid_with_roof(nv, where):
    """nv vertices (those the grid has no use for lie on it), triangles; the roof is the last triangle."""
    k = 8
    xy = np.stack(np.meshgrid(np.linspace(-1, 1, k), np.linspace(-1, 1, k), indexing="ij"), -1).reshape(-1, 2)
    grid = np.concatenate([xy, np.zeros((k * k, 1))], 1)
    spare = np.zeros((nv - k * k - 3, 3))
    spare[:, :2] = np.random.default_rng(1).uniform(-1, 1, (len(spare), 2))
    roof = np.array([[-0.9, -0.9, 0.4], [0.9, -0.9, 0.4], [0.0, 0.9, 0.4]])
    flat = np.concatenate([grid, spare])
    at = {"first": 0, "middle": len(flat) // 2, "last": len(flat)}[where]
    V = np.concatenate([flat[:at], roof, flat[at:]]).astype(np.float32)
    new = np.arange(len(flat)) + np.where(np.arange(len(flat)) >= at, 3, 0)
    i, j = np.meshgrid(np.arange(k - 1), np.arange(k - 1), indexing="ij")
    a = (i * k + j).ravel()
    T = np.concatenate([np.stack([a, a + k, a + k + 1], 1), np.stack([a, a + k + 1, a + 1], 1)])
    return V, np.concatenate([new[T], [[at, at + 1, at + 2]]]).astype(np.uint32)


@pytest.mark.parametrize("where", ["first", "middle", "last"])
@pytest.mark.parametrize("nv", [70, 255, 257, 1023, 1024, 1025, 5000])
def test_a_roof_is_seen_from_below(nv, where):
    from paper_1312_3691_amd import tpmc
    V, T = _grid_with_roof(nv, where)
    assert len(V) == nv
    q = I.query(q=tuple(I.quat_for_flow((0.6, 0.0, -0.8))), S=3.0, n=40_000, seed=5, alpha=1.0)
    o = O.run(V, T, q, A_ref=1.0)
    ctx = tpmc.Context(0)
    for builder in ("sah", "lbvh"):
        mesh = ctx.build_mesh(V, T, builder=builder)
        res, pr = tpmc.run(mesh, [q], A_ref=1.0)
        counts = pr.tally(0)[:, 6]
        pr.close()
        mesh.close()
        assert abs(res[0]["hits"] - o["hits"]) <= 1e-3 * o["hits"] + 3, builder
        assert abs(counts[-1] - o["tri"][-1, 6]) <= 1e-3 * o["hits"] + 3, builder
        assert o["hits"] - (q["n"] - o["missed"]) > 0.03 * o["hits"]  # what would be lost: hits after the first
