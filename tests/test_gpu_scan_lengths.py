"""The per-phase rounds' scans at lengths of one workgroup, of several, and of
more than 2048 (where the workgroups' totals are scanned by a launch of their
own): plan store, counters and result equal those of the single launch, whose
scans are another code."""

import numpy as np
import pytest

from paper_1607_06886_amd import scenes
from tests._gpu import planner_for, print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r_conn,least_pairs", [(40, 1.0, 0), (700, 1.0, 1024), (2600, 4.0, 2049 * 1024)])
def test_rounds_per_phase_equal_the_single_launch(n, r_conn, least_pairs):
    print_case("scan lengths", n=n, r_conn=r_conn)
    sc = scenes.make_scene(dict(n=n, n_obs=2, side=(0.1, 0.2), N=32, sigma=0.02, alpha=0.2, indoor=False),
                           23, M=256, S_max=128)
    pl = planner_for(sc, dt=0.2, r_conn=r_conn, cap_pairs=1 << 23)
    pr = pl.scene_problem(sc, device=True)
    got = []
    for mode in (1, 0):
        pl.set_explore_mode(mode)
        r = pl.plan(pr)
        got.append((r, pl.plans()))
    (r1, s1), (r0, s0) = got
    for k in s1:
        np.testing.assert_array_equal(s1[k], s0[k], err_msg=k)
    for k in ("status", "rounds", "partial_plans", "simulated", "preprune", "inserted", "n_plans", "best_cost"):
        assert r1[k] == r0[k], k
    print("  pairs", r0["partial_plans"], "rounds", r0["rounds"], flush=True)
    assert r0["partial_plans"] >= least_pairs * r0["rounds"]   # (some round is that long)
    pl.close()
