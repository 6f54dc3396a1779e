"""The kernel with a search in every lane, at row widths and frame sizes
where its parts meet: frames longer than the LDS copy, stacks that go on in
the wavefront's worst-case area, rows of each width, both directions.

With the incumbent held at the optimum (goal = optimum + 1) every search
order evaluates the same nodes, so counts must equal the oracle's: a frame
lost or done twice when lanes or wavefronts hand work on changes them."""
import math

import numpy as np
import pytest

import mcs_instances as mi
import oracle

pytestmark = pytest.mark.gpu


def _labelled(rng, n, p, directed, share):
    nlab = max(1, math.ceil(share * n))
    return tuple(mi.random_small(rng, n, p, directed, nlab) for _ in range(2))


# (n lowest, n highest, p, labels per vertex): 32-, 64-, 128- and 256-bit rows
SHAPES = [(28, 32, 0.2, 0.2), (33, 64, 0.1, 0.5), (65, 110, 0.1, 0.8), (129, 200, 0.5, 0.8)]


def _case(shape, directed):
    from _mcsplit_py import rank, root, select
    n0, n1, p, share = shape
    rng = np.random.default_rng([n0, directed])
    pairs, goals, counts = [], [], []
    for k in range(40):
        n = n1 if k == 0 else int(rng.integers(n0, n1 + 1))
        G, H = _labelled(rng, n, p, directed, share)
        o = oracle.mcs(G, H, node_limit=3_000_000)
        classes = root(G, H)
        if not o["complete"] or not classes:
            continue
        rg = rank(G)
        v0 = min(classes[select(classes, rg)][0], key=lambda x: rg[x])
        pairs.append((G, H))
        goals.append(o["size"] + 1)
        counts.append(oracle.branch_cost(G, H, [], v0, o["size"]))
        if len(pairs) == 12:
            break
    return pairs, goals, counts


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_node_counts_under_a_fixed_incumbent(gpu, shape, directed):
    from paper_1908_06418_amd import Plan
    pairs, goals, counts = _case(shape, directed)
    assert len(pairs) >= 4 and max(max(G["n"], H["n"]) for G, H in pairs) > shape[0]
    for tun in ({}, {"check_interval": 1, "donate_low": 64, "ring_slots": 64, "waves_per_cu": 1}):
        print(f"lane kernel, {shape}, directed {directed}, {tun}: {len(pairs)} pairs", flush=True)
        plan = Plan(pairs, time_limit_s=60, tuning=tun).upload()
        try:
            plan.set_goals(goals)
            plan.run()
            res = plan.results()
        finally:
            plan.close()
        assert all(r.optimal and r.size < g for r, g in zip(res, goals))
        assert [r.nodes for r in res] == counts


@pytest.mark.parametrize("directed", [False, True])
def test_deep_stacks_go_on_in_the_worst_case_area(gpu, directed):
    """Relabelled copies of sparse 60- to 64-vertex graphs: a search dives
    through up to n frames of up to n classes, more than one lane's part of
    the stack holds."""
    from paper_1908_06418_amd import Plan
    rng = np.random.default_rng(5)
    pairs = []
    for n in (60, 63, 64):
        G = mi.random_small(rng, n, 0.15, directed)
        pairs.append((G, mi.permute(G, [int(x) for x in rng.permutation(n)])))
    plan = Plan(pairs, time_limit_s=60).upload()
    try:
        plan.run()
        res = plan.results()
        st = plan.stats()
    finally:
        plan.close()
    for (G, H), r in zip(pairs, res):
        assert r.optimal and r.size == G["n"]
        assert oracle.check.is_valid(G, H, r.mapping)
    assert st.hbm_frames > 0


@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("shape,directed,depth", [((28, 32, 0.2, 0.2), False, 1),
                                                  ((28, 32, 0.2, 0.2), True, 8),
                                                  ((33, 64, 0.1, 0.5), False, 3),
                                                  ((33, 64, 0.1, 0.5), True, 0)])
def test_learned_order_keeps_every_size(gpu, shape, directed, depth, mode):
    """The learned order, whose shallow frames hold their partners' order
    beside the stack: it changes neither the proven size nor, with the order
    of the partners alone and the incumbent fixed, the number of nodes."""
    from paper_1908_06418_amd import Plan
    from paper_1908_06418_amd.policy import Policy
    pairs, goals, counts = _case(shape, directed)
    P = Policy(seed=31)
    for tun in ({}, {"check_interval": 1, "donate_low": 64, "ring_slots": 64, "waves_per_cu": 1}):
        print(f"learned lane kernel, {shape}, directed {directed}, depth {depth}, mode {mode}, "
              f"{tun}: {len(pairs)} pairs", flush=True)
        plan = Plan(pairs, time_limit_s=60, tuning=tun, policy=P, policy_depth=depth,
                    policy_mode=mode).upload()
        try:
            plan.run()
            assert [r.size + 1 for r in plan.results()] == goals
            for r, (G, H) in zip(plan.results(), pairs):
                assert r.optimal and oracle.check.is_valid(G, H, r.mapping)
            plan.set_goals(goals)
            plan.run()
            res = plan.results()
            assert all(r.optimal and r.size + 1 == g or r.size == 0 for r, g in zip(res, goals))
            if mode == 2:
                assert [r.nodes for r in res] == plain_counts(pairs, goals)
        finally:
            plan.close()


def plain_counts(pairs, goals):
    from paper_1908_06418_amd import Plan
    plan = Plan(pairs, time_limit_s=60).upload()
    plan.set_goals(goals)
    plan.run()
    out = [r.nodes for r in plan.results()]
    plan.close()
    return out
