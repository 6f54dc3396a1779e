"""The learned order in the lane kernel against the float64 features of
oracle.policy: which v it picks, in which order it tries the partners, and
that it changes nothing else."""
import numpy as np
import pytest
from _mcsplit_py import Counter, rank, root
from test_gpu_lane import _case
from test_gpu_policy import _feature_net

import mcs_instances as mi
import oracle
from oracle import policy as ref

pytestmark = pytest.mark.gpu

VARYING = (0, 5, 6, 7, 8, 9, 13)


def _pairs(directed, labels):
    rng = np.random.default_rng([21, directed, labels])
    out = []
    for _ in range(10):
        n, p = int(rng.integers(11, 16)), float(rng.uniform(0.2, 0.6))
        out.append(tuple(mi.random_small(rng, n, p, directed, labels) for _ in range(2)))
    return out


@pytest.mark.parametrize("directed,labels", [(False, 0), (False, 2), (True, 0)])
def test_choice_of_v(gpu, directed, labels):
    """With the incumbent held at the optimum the nodes depend on the choices
    of v alone: they are those of the Python recursion that takes the vertex
    of the highest (or lowest) feature k at |M| <= 3."""
    from paper_1908_06418_amd import Plan
    from paper_1908_06418_amd.policy import Policy
    pairs = _pairs(directed, labels)
    goals = [oracle.mcs(G, H)["size"] + 1 for G, H in pairs]
    seen = set()
    for k in VARYING:
        for sign in (1.0, -1.0):
            want = []
            for (G, H), g in zip(pairs, goals):
                def score(u, side, classes, sel, d, cand, G=G):
                    return sign * round(ref.features(G, u, side, classes, sel, d, cand)[k] * G["n"])
                c = Counter(G, H, g - 1, score=score, depth_max=3, mode=1)
                c.rec(root(G, H), 0)
                want.append(c.nodes)
            print(f"lane scorer, directed {directed}, labels {labels}, feature {k}, {sign:+.0f}",
                  flush=True)
            plan = Plan(pairs, time_limit_s=60, policy=Policy(params=_feature_net(k, sign)),
                        policy_depth=3, policy_mode=1).upload()
            try:
                plan.set_goals(goals)
                plan.run()
                res = plan.results()
            finally:
                plan.close()
            assert all(r.optimal and r.size < g for r, g in zip(res, goals))
            assert [r.nodes for r in res] == want, (k, sign)
            seen.add(tuple(want))
    assert len(seen) >= 7  # the orders really differ


@pytest.mark.parametrize("k", range(ref.F))
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_order_of_the_partners_at_the_root(gpu, k, sign):
    """The order that the root's frame keeps in the workspace, for whichever v
    it was made last: the partners by feature k, ties to the earlier one."""
    import torch
    from paper_1908_06418_amd import Plan
    from paper_1908_06418_amd.policy import Policy
    rng = np.random.default_rng(33)
    G, H = (mi.random_small(rng, 22, 0.3) for _ in range(2))
    r = rank(H)
    every = sorted(range(H["n"]))
    patterns = set()
    for left in range(1, G["n"] + 1):
        classes = [(set(range(left)), set(every))]
        s = {u: sign * round(ref.features(H, u, 1, classes, 0, 0, every)[k] * H["n"])
             for u in every}
        patterns.add(bytes(r[u] for u in sorted(every, key=lambda u: (-s[u], r[u]))))
    print(f"lane scorer, partners by feature {k}, {sign:+.0f}: {len(patterns)} orders", flush=True)
    plan = Plan([(G, H)], time_limit_s=60, tuning={"use_graph": 1, "waves_per_cu": 1},
                policy=Policy(params=_feature_net(k, sign)), policy_depth=0, policy_mode=2).upload()
    try:
        plan.ws.zero_()  # (the graph copies the inputs in)
        torch.cuda.synchronize()
        plan.run()
        res = plan.results()
        memory = plan.ws.cpu().numpy().tobytes()
    finally:
        plan.close()
    assert res[0].optimal and res[0].size == oracle.mcs(G, H)["size"]
    assert any(p in memory for p in patterns)


@pytest.mark.parametrize("mode,depth", [(1, 3), (2, 4), (3, 2)])
@pytest.mark.parametrize("shape,directed", [((28, 32, 0.2, 0.2), False), ((33, 64, 0.1, 0.5), True)])
def test_sizes_and_counts_are_the_oracles(gpu, shape, directed, mode, depth):
    """The deepest orders that the lane kernel takes.  Ordering the partners
    alone, under a fixed incumbent, leaves the oracle's node counts."""
    from paper_1908_06418_amd import Plan
    from paper_1908_06418_amd.policy import Policy
    pairs, goals, counts = _case(shape, directed)
    print(f"lane scorer, {shape}, directed {directed}, mode {mode}, depth {depth}", flush=True)
    plan = Plan(pairs, time_limit_s=60, policy=Policy(seed=31), policy_depth=depth,
                policy_mode=mode).upload()
    try:
        plan.run()
        res = plan.results()
        assert all(r.optimal for r in res) and [r.size + 1 for r in res] == goals
        plan.set_goals(goals)
        plan.run()
        res = plan.results()
    finally:
        plan.close()
    assert all(r.optimal and r.size < g for r, g in zip(res, goals))
    if mode == 2:
        assert [r.nodes for r in res] == counts
