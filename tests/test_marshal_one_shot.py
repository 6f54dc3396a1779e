"""Labels that can be gone through only once, beside a graph that the flat
marshalling does not take: they are read once."""
import numpy as np
import pytest

import mcs_instances as mi


class _Once:
    """One pass, by a fresh iterator each time."""

    def __init__(self, xs):
        self.it = iter(xs)

    def __iter__(self):
        return (x for x in self.it)


@pytest.mark.parametrize("once", [lambda xs: map(int, xs), iter, _Once, lambda xs: (x for x in xs)])
@pytest.mark.parametrize("other", [{"n": 3, "directed": False, "rows": np.array([2.0, 1.0, 0.0]),
                                    "label": None},
                                   {"n": 3, "directed": False, "rows": [2, 1, 0],
                                    "label": np.array([1.0, 2.0, 3.0])}, mi.er_graph(5, 0.5, 1)])
def test_one_shot_labels_are_read_once(once, other):
    from paper_1908_06418_amd import _Marshal
    g = {"n": 3, "directed": False, "rows": [2, 1, 0], "label": once([7, 8, 9])}
    h = {"n": 3, "directed": False, "rows": [0, 0, 0], "label": once([5, 6, 4])}
    m = _Marshal([(g, h), (other, other)])
    assert [m.G[0].label[k] for k in range(3)] == [7, 8, 9]
    assert [m.H[0].label[k] for k in range(3)] == [5, 6, 4]
