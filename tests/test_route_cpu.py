"""Which kernel a plan takes under the knobs that change it, seen by its
workspace: each kernel lays it out its own way."""
import numpy as np
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


def _copies(n, p, count, directed=False, labels=0):
    rng = np.random.default_rng([n, directed])
    gs = [mi.random_small(rng, n, p, directed, labels) for _ in range(count)]
    return [(g, mi.permute(g, [int(x) for x in rng.permutation(n)])) for g in gs]


def _flipped(pair):
    g, h = pair
    rows = list(h["rows"])
    rows[3] ^= 1 << 7
    rows[7] ^= 1 << 3
    return g, dict(h, rows=rows)


def _random(n, count):
    rng = np.random.default_rng(n)
    return [tuple(mi.random_small(rng, n, 0.2) for _ in range(2)) for _ in range(count)]


EMPTY = [(mi.er_graph(50, 0.0, 1), mi.er_graph(50, 0.0, 2))]


@pytest.mark.parametrize("pairs,lane", [
    (_copies(64, 0.2, 2), False), (_copies(34, 0.2, 1), False), (_copies(40, 0.15, 2, True), False),
    ([_flipped(p) for p in _copies(48, 0.2, 3)], False), (EMPTY, False), (_copies(32, 0.2, 2), True),
    (_copies(28, 0.2, 2, True), False), (_copies(20, 0.3, 2, False, 6), False),
    (_random(40, 2), True), (_random(64, 1), True), (_copies(40, 0.2, 2) + _random(40, 1), True)])
def test_copies_with_long_frames_are_not_for_one_search_in_every_lane(mcs_lib, pairs, lane):
    from paper_1908_06418_amd import workspace_size
    segments = workspace_size(pairs, tuning={"seg_lanes": 8})
    assert (workspace_size(pairs) != segments) is lane


@pytest.mark.parametrize("mode,deepest", [(1, 3), (2, 4), (3, 2)])
def test_deep_learned_orders_are_not_for_one_search_in_every_lane(mcs_lib, mode, deepest):
    import ctypes

    import torch

    from paper_1908_06418_amd import _Marshal, _opts
    params = torch.zeros(6000, dtype=torch.float16)  # (only its address is taken)
    aligned = params[(-params.data_ptr() % 16) // 2:]
    m = _Marshal(SMALL)
    for depth in range(9):
        size = [int(mcs_lib.mcs_workspace_size(len(SMALL), m.G, m.H, ctypes.byref(
            _opts(0, 0, tun, policy=aligned, policy_depth=depth, policy_mode=mode)[0])))
            for tun in (None, {"seg_lanes": 64})]
        assert (size[0] != size[1]) is (depth <= deepest)


@pytest.mark.parametrize("waves", [0, 1, 2, 3])
def test_few_wavefronts_fit_the_largest_workgroup(mcs_lib, waves):
    """(Without a device the plan assumes workgroups of 64 KiB of LDS.)"""
    from paper_1908_06418_amd import workspace_size
    rng = np.random.default_rng(12)
    for n, labels in ((70, 50), (129, 100), (254, 180)):
        pairs = [tuple(mi.random_small(rng, n, 0.3, True, labels) for _ in range(2))]
        assert workspace_size(pairs, tuning={"waves_per_cu": waves}) > 0
