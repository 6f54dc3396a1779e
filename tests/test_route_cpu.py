"""Which kernel a plan takes under the knobs that change it, seen by its
workspace: each kernel lays it out its own way."""
import pytest

import mcs_instances as mi

SMALL = [(mi.er_graph(20, 0.3, 2 * k + 1), mi.er_graph(20, 0.3, 2 * k + 2)) for k in range(3)]
WIDE = [(mi.er_graph(70, 0.1, 2 * k + 1, True, True), mi.er_graph(70, 0.1, 2 * k + 2, True, True))
        for k in range(3)]


@pytest.mark.parametrize("pairs,seg", [(SMALL, 8), (WIDE, 64)])
def test_never_donating_is_not_for_one_search_in_every_lane(mcs_lib, pairs, seg):
    from paper_1908_06418_amd import workspace_size
    assert workspace_size(pairs, tuning={"donate_low": -1}) == \
        workspace_size(pairs, tuning={"donate_low": -1, "seg_lanes": seg})
    assert workspace_size(pairs, tuning={"donate_low": 1}) != \
        workspace_size(pairs, tuning={"donate_low": 1, "seg_lanes": seg})
