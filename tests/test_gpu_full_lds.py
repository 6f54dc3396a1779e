"""A plan whose workgroup takes all the LDS that is left beside the kernel's
copy of its parameters."""
import numpy as np
import pytest

import mcs_instances as mi
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [1, 4])
def test_a_workgroup_that_fills_lds(gpu, waves):
    """Directed pairs of 33 and up to 56 vertices, 16-lane segments: 163,584
    bytes of LDS in a workgroup, of 163,840."""
    from paper_1908_06418_amd import Plan
    rng = np.random.default_rng(6)
    pairs = [(mi.random_small(rng, 33, 0.1, True, 24), mi.random_small(rng, n, 0.1, True, 24))
             for n in (56, 40, 33)]
    plan = Plan(pairs, time_limit_s=30, tuning={"seg_lanes": 16, "waves_per_cu": waves}).upload()
    try:
        plan.run()
        res = plan.results()
        st = plan.stats()
    finally:
        plan.close()
    assert st.lds_per_wave == 40896
    for (G, H), r in zip(pairs, res):
        assert r.optimal and r.size == oracle.mcs(G, H)["size"]
        assert oracle.check.is_valid(G, H, r.mapping)
