"""Nodes of the lane kernel under a node limit or a dead-end forecast, which
wavefronts hand in by the thousand as they go."""
import pytest
from test_gpu_lane import SHAPES, _case

import mcs_instances as mi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limits", [{"node_limit": 10 ** 15}, {"deadend_nodes": 10 ** 12},
                                    {"node_limit": 10 ** 15, "deadend_nodes": 10 ** 12}])
@pytest.mark.parametrize("shape", SHAPES)
def test_counts_under_limits_that_are_never_met(gpu, shape, limits):
    from paper_1908_06418_amd import Plan
    pairs, goals, counts = _case(shape, False)
    for tun in ({}, {"check_interval": 1, "waves_per_cu": 1}, {"check_interval": 300}):
        print(f"lane limits, {shape}, {limits}, {tun}: {len(pairs)} pairs", flush=True)
        plan = Plan(pairs, time_limit_s=60, tuning=tun, **limits).upload()
        try:
            plan.set_goals(goals)
            plan.run()
            res = plan.results()
            st = plan.stats()
        finally:
            plan.close()
        assert st.stopped == 0 and all(r.optimal and r.size < g for r, g in zip(res, goals))
        assert [r.nodes for r in res] == counts


@pytest.mark.parametrize("limit", [1, 3_000_000, 200_000_000])
def test_a_node_limit_stops_soon_after(gpu, limit):
    """A wavefront may hold back 999 nodes and those of four steps (64 lanes,
    at most two partners and three unmatched children each: 1,280), and it
    hears of the stop up to some 10 us later, a few more steps."""
    from paper_1908_06418_amd import Plan
    pairs = mi.pairs_c2(ns=(35,), ps=(0.3,), seeds=range(3))
    print(f"lane limits, stop after {limit} nodes", flush=True)
    plan = Plan(pairs, node_limit=limit, time_limit_s=60).upload()
    try:
        plan.run()
        res = plan.results()
        st = plan.stats()
    finally:
        plan.close()
    assert st.stopped == 1 and not any(r.optimal for r in res)
    assert limit <= sum(r.nodes for r in res) == st.nodes <= limit + 8000 * st.waves


@pytest.mark.parametrize("limit", [1000, 20_000, 200_000, 2_000_000])
@pytest.mark.parametrize("seeds", [1, 10])
def test_small_node_limits_are_met_closely(gpu, limit, seeds):
    """A small limit is looked at after every step, with next to nothing held
    back: what comes on top is the step that each wavefront is in, and while
    a search spreads, its lanes double at most from one step to the next (so
    twice the limit, and again what starts before the stop is seen)."""
    from paper_1908_06418_amd import Plan
    pairs = mi.pairs_c2(ns=(35,), ps=(0.3, 0.5), seeds=range(seeds))
    print(f"lane limits, {len(pairs)} pairs, {limit} nodes", flush=True)
    plan = Plan(pairs, node_limit=limit, time_limit_s=60).upload()
    try:
        plan.run()
        st = plan.stats() if plan.results() else None
    finally:
        plan.close()
    assert st.stopped == 1 and limit <= st.nodes <= 4 * limit + 1000
