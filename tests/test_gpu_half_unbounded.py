"""The half-space model where the particle cloud has no bound on an axis: a
plane at a right angle to that axis has no reach that could rule it out (0
times infinity), and the other particles beyond it count all the same.

Nodes and velocities lie in a plane z = const, so walls that pass through it
have planes at a right angle to z, and the ceiling's plane marks every waypoint
at which some particle's z is infinite.  One pair of particles after the other
gets infinite normals of either sign on z (infinite for a step or two, then
NaN), so the cloud is unbounded to both sides at every early step."""

import numpy as np
import pytest

from paper_1607_06886_amd import scenes
from tests._gpu import planner_for, print_case
from tests.test_gpu_half_batches import _check

pytestmark = pytest.mark.gpu

Z = np.float32(0.3)


def _scene(N):
    sc = scenes.make_scene(dict(n=260, n_obs=3, side=(0.1, 0.3), N=N, sigma=0.05, alpha=0.6, indoor=False),
                           77, M=256, S_max=160)
    sc.samples[:, 2], sc.samples[:, 5] = Z, 0.0
    sc.x_init[2], sc.x_init[5] = Z, 0.0
    sc.goal[2], sc.goal[5] = 0.2, 0.4
    sc.obstacles = np.array([[0.25, 0.0, 0.0, 0.3, 0.4, 0.5],       # two walls
                             [0.0, 0.55, 0.0, 0.45, 0.6, 0.5],
                             [0.0, 0.0, 0.6, 1.0, 1.0, 0.7]],        # the ceiling
                            np.float32)
    for j in range(N // 4):                                          # particles 0 .. N/2 - 1
        sc.noise[3 + j, 4, j] = np.inf
        sc.noise[3 + j, 4, N // 4 + j] = -np.inf
    return sc


@pytest.mark.parametrize("N", [32, 128])
def test_planes_beside_an_unbounded_cloud(N):
    print_case("half-space, unbounded cloud", N=N)
    sc = _scene(N)
    pl = planner_for(sc, cp_model=1)
    pr = pl.scene_problem(sc, device=True)
    for mode in (0, 1):
        pl.set_explore_mode(mode)
        pl.plan(pr)
        D = pl.deviation()
        for sign in (np.inf, -np.inf):
            assert (D[4:4 + N // 4, 2] == sign).any(axis=1).all()
        st = pl.plans()
        with np.errstate(invalid="ignore"):
            n, _ = _check(st, pl.graph(sc.n + 1), sc, D, 200)
        bits = np.unpackbits(st["mask"].view(np.uint8), axis=1, bitorder="little").astype(bool)
        wall_hits = int(bits[:, N // 2:].sum())    # particles that are finite throughout
        print("  plans", n, "hits of finite particles", wall_hits, flush=True)
        assert n > 20 and wall_hits > 0
    pl.close()
