"""Queries packed and results unpacked at once against the structures' own
fields: equal bytes, equal values and types, the same refusals."""
import ctypes

import numpy as np
import pytest

from paper_1312_3691_amd import inputs as I
from paper_1312_3691_amd import tpmc


def _dicts():
    base = dict(q=(1, 0, 0, 0), S=5, T_inf=1000, T_w=300.0, alpha=1, n=1000, seed=1)
    return [base, dict(base, q=np.array([0.5, 0.5, -0.5, 0.5]), S=np.float32(3.3), n=np.int64(1 << 40), seed=-1),
            dict(base, n=1e6, seed=2 ** 64 + 5, flags=2 ** 32 + 7, max_reflections=-1, cv_center=np.arange(3.0),
                 cv_radius=2, alpha_E=0.5), dict(base, S=float("nan"), T_w="300", n=True), dict(base, n=-3)
            ] + [I.query(q=tuple(q), S=0.1, n=7, seed=i, cv_box=bool(i % 2)) for i, q in enumerate(I.random_quats(3, 1))]


def test_packed_queries_equal_the_structures():
    ds = _dicts()
    arr = tpmc._queries(ds)
    assert isinstance(arr[0], tpmc.Query) and len(arr) == len(ds)
    for d, q in zip(ds, arr):
        assert bytes(q) == bytes(tpmc.make_query(d)), d
    assert len(tpmc._queries([])) == 0


@pytest.mark.parametrize("bad", [dict(q=(1, 0, 0)), dict(q=(1, 0, 0, 0, 0)), dict(cv_center=(0, 0)), dict(S=None),
                                 dict(n="x"), dict(seed=None), dict(alpha=1j)])
def test_refused_by_both(bad):
    d = dict(_dicts()[0], **bad)
    kinds = []
    for f in (tpmc.make_query, lambda d: tpmc._queries([d])):
        with pytest.raises((ValueError, TypeError)) as e:
            f(d)
        kinds.append(e.type)
    assert kinds[0] is kinds[1]


@pytest.mark.parametrize("n", [0, 1, 7, 8, 9])
def test_results_equal_the_structures(n):
    raw = np.random.default_rng(n).bytes(n * ctypes.sizeof(tpmc.Result))
    res = (tpmc.Result * n).from_buffer_copy(raw)
    got = tpmc.result_dicts(res)
    assert len(got) == n
    for g, r in zip(got, res):
        w = {f: getattr(r, f) for f, _ in tpmc.Result._fields_}
        w = {f: np.array(v[:]) if isinstance(v, ctypes.Array) else v for f, v in w.items()}
        assert list(g) == list(w)
        for k in w:
            assert type(g[k]) is type(w[k]), k
            assert np.array_equal(np.asarray(g[k]), np.asarray(w[k]), equal_nan=np.asarray(w[k]).dtype == float), k
            if isinstance(w[k], np.ndarray):
                assert g[k].dtype == w[k].dtype and g[k].flags.writeable and g[k].flags.owndata
