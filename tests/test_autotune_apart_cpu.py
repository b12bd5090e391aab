"""The tuner measures a launch once: values of groups_per_cu at or above what a
compute unit holds give the same launch.  No GPU."""
from paper_1312_3691_amd import autotune as AT


def test_groups_beyond_the_resident_ones_are_one_setting():
    tried = []

    def cost(t):
        tried.append(t["groups_per_cu"])
        return 1.0

    axes = AT.launched_apart(AT.free_axes(None), AT.DEFAULT)
    AT.coordinate_search(cost, axes=axes)
    assert set(tried) == {AT.DEFAULT["groups_per_cu"]}
    assert [n for n, _ in axes] == [n for n, _ in AT.AXES]
    for name, values in axes[:2]:
        assert values == dict(AT.AXES)[name]
    # from a start below, one value launches what the start does not
    low = AT.launched_apart(AT.AXES, dict(AT.DEFAULT, groups_per_cu=2))
    assert dict(low)["groups_per_cu"] == [4]
