"""The lane kernel on pairs whose searches run through their lane's part of the
stack into the wavefront's worst-case area, many of them at once: with the
incumbent held at the optimum the node counts must be the oracle's."""
import math

import numpy as np
import pytest

import mcs_instances as mi
import oracle

pytestmark = pytest.mark.gpu


# n lowest, n highest, p, labels per vertex, directed: a single search in
# sequential order holds 210 to 350 entries at its deepest on the first kind
# (a lane's part: 160), 170 to 220 on the second, 380 to 650 on the third (256)
@pytest.mark.parametrize("n0,n1,p,share,directed", [(60, 64, 0.05, 0.6, False),
                                                    (60, 64, 0.05, 0.6, True),
                                                    (100, 128, 0.05, 0.9, False)])
def test_node_counts_through_the_worst_case_area(gpu, n0, n1, p, share, directed):
    from _mcsplit_py import rank, root, select

    from paper_1908_06418_amd import Plan
    rng = np.random.default_rng([n0, directed, 3])
    pairs, goals, counts = [], [], []
    for _ in range(14):
        n = int(rng.integers(n0, n1 + 1))
        G, H = (mi.random_small(rng, n, p, directed, max(1, math.ceil(share * n)))
                for _ in range(2))
        o = oracle.mcs(G, H, node_limit=3_000_000)
        if not o["complete"]:
            continue
        classes = root(G, H)
        rg = rank(G)
        v0 = min(classes[select(classes, rg)][0], key=lambda x: rg[x])
        pairs.append((G, H))
        goals.append(o["size"] + 1)
        counts.append(oracle.branch_cost(G, H, [], v0, o["size"]))
    assert len(pairs) >= 5
    for tun in ({}, {"check_interval": 1, "donate_low": 64, "ring_slots": 64, "waves_per_cu": 1}):
        print(f"worst-case area, {n0}-{n1}, directed {directed}, {tun}: {len(pairs)} pairs",
              flush=True)
        plan = Plan(pairs, time_limit_s=60, tuning=tun).upload()
        try:
            plan.set_goals(goals)
            plan.run()
            res = plan.results()
            st = plan.stats()
        finally:
            plan.close()
        assert st.hbm_frames > 0
        assert all(r.optimal and r.size < g for r, g in zip(res, goals))
        assert [r.nodes for r in res] == counts
