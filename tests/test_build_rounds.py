"""Bodies whose SAH build takes more levels than are enqueued before the host first
looks (build_bvh_sah goes round again), or has a big node that no plane separates
(handed to the mid stage as it is).  A replay of the binned splits on the CPU says
which body does what; on the GPU the results, per-triangle loads and first hits
equal those on the LBVH bit for bit."""
import math

import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I

BIG, WAVE, BINS, MAX_LEVEL = 1024, 32, 32, 32  # csrc/tpmc_bvh.hip, csrc/tpmc_sah.hpp


def _graded(n, octaves, seed):
    """n triangles whose centres crowd towards the origin, as many in each octave, their sizes with them."""
    r = np.random.default_rng(seed)
    c = r.uniform(0.5, 1.0, (n, 3)) * 2.0 ** -(np.arange(n) % octaves)[:, None]
    V = c[:, None, :] * (1.0 + r.normal(0, 0.02, (n, 3, 3)))
    return r.permutation(V.astype(np.float32)).reshape(-1, 3), np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)


def _copies(n):
    V = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0.5]], dtype=np.float32)
    return V, np.tile(np.arange(3, dtype=np.uint32), (n, 1))


# name: body, big levels beyond the first burst, mid levels beyond it, unbinnable big nodes
BODIES = {"graded20000": (_graded(20_000, 60, 1), True, False, False),
          "graded1000": (_graded(1_000, 60, 2), False, True, False),
          "graded3000": (_graded(3_000, 60, 4), True, True, False),
          "copies5000": (_copies(5_000), False, False, True),
          "copies60000": (_copies(60_000), False, True, True)}


def _levels_to(n, to):
    levels = 0
    while n > to:
        n, levels = (n + 1) // 2, levels + 1
    return levels


def _replay(V, T):
    """(levels of the big stage, of the mid stage, unbinnable big nodes) of a body's build."""
    P = V[T.astype(np.int64)]
    lo, hi = P.min(1), P.max(1)
    c = np.float32(0.5) * (lo + hi)
    big = mid = unbinned = 0
    work = [(np.arange(len(T)), 0, 0)]  # triangles, tree level, mid levels above it
    while work:
        t, level, above = work.pop()
        m = len(t)
        if m <= WAVE:
            continue
        best = (math.inf, None)
        for k in range(3):
            x = c[t, k]
            ext = x.max() - x.min()
            if level >= MAX_LEVEL or not ext > 0:
                continue
            b = np.minimum(BINS - 1, ((x - x.min()) * (np.float32(BINS) / ext)).astype(np.int64))
            for plane in range(1, BINS):
                left = b < plane
                if not left.any() or left.all():
                    continue
                cost = 0.0
                for side in (left, ~left):
                    e = (hi[t[side]].max(0) - lo[t[side]].min(0)).astype(np.float64)
                    cost += (e[0] * e[1] + e[1] * e[2] + e[2] * e[0]) * side.sum()
                if cost < best[0]:
                    best = (cost, left)
        left = best[1]
        if m > BIG and above == 0:
            big = max(big, level + 1)
            if left is None:
                unbinned += 1
        in_mid = above > 0 or m <= BIG or left is None
        if in_mid:
            mid = max(mid, above + 1)
        if left is None:
            left = np.arange(m) < m // 2
        for side in (left, ~left):
            work.append((t[side], level + 1, above + 1 if in_mid else 0))
    return big, mid, unbinned


@pytest.mark.parametrize("name", sorted(BODIES))
def test_bodies_take_the_branches(name):
    (V, T), more_big, more_mid, unbinnable = BODIES[name]
    n = len(T)
    big_burst = _levels_to(n, BIG) * 3 // 2 + 1 if n > BIG else 0
    mid_burst = _levels_to(min(n, BIG), WAVE) * 3 // 2 + 2
    big, mid, unbinned = _replay(V, T)
    assert (big > big_burst, mid > mid_burst, unbinned > 0) == (more_big, more_mid, unbinnable), \
        (big, big_burst, mid, mid_burst, unbinned)


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(BODIES))
def test_sah_equals_lbvh(name):
    from paper_1312_3691_amd import tpmc
    ctx = tpmc.Context(0)
    V, T = BODIES[name][0]
    q = I.query(S=3.0, n=2_001, seed=8, alpha=0.9, q=tuple(I.random_quats(1, 4)[0]))
    got = {}
    for builder in ("sah", "lbvh"):
        mesh = ctx.build_mesh(V, T, builder=builder)
        assert 1 <= mesh.info["depth"] <= 64
        res, pr = tpmc.run(mesh, [q], A_ref=1.0, first_tri=True)
        got[builder] = (res[0], pr.tally(), pr.first_tri.cpu().numpy())
        pr.close()
        mesh.close()
    a, b = got["sah"], got["lbvh"]
    assert a[0]["guard_trips"] == 0 and b[0]["guard_trips"] == 0 and a[0]["hits"] > 0
    for k in tpmc.same_on_every_path(a[0]):
        assert np.array_equal(np.asarray(a[0][k]), np.asarray(b[0][k])), (name, k)
    assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
