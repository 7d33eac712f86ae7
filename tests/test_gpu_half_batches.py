"""The half-space model's expansion (headers, then batches of queued pairs with
their planes in LDS): each plan's bits are its parent's and those of the
particles beyond some plane of some waypoint's region (oracle/hsmc.py), from the
library's own deviation table.  Every particle count, box sets of none to three
64-bit words, clouds wide enough that a batch's planes overrun their pool, and
both ways to run the rounds (a launch per phase: short batches; one launch).

A particle within 1e-9 of a plane is left out: nominal points of order 1 differ
by some 1e-15 between the two sides, and so do the planes."""

import numpy as np
import pytest

from oracle import hsmc
from paper_1607_06886_amd import scenes
from tests._gpu import planner_for, print_case

pytestmark = pytest.mark.gpu

DT = float(np.float32(0.05))


def _check(st, g, sc, D, limit):
    X = np.concatenate([sc.x_init[None], sc.samples]).astype(np.float64)
    bits = np.unpackbits(st["mask"].view(np.uint8), axis=1, bitorder="little").astype(bool)
    boxes = sc.obstacles.astype(np.float64)
    order = np.random.default_rng(0).permutation(np.arange(1, len(st["head"])))[:limit]
    hits = 0
    for p in order:
        q, e = st["parent"][p], st["edge"][p]
        x0, x1, tau = X[st["head"][q]], X[st["head"][p]], g["tau"][e]
        P, v0, v1 = x1[:3] - x0[:3], x0[3:], x1[3:]
        c2 = (3 * P - (2 * v0 + v1) * tau) / tau ** 2
        c3 = (-2 * P + (v0 + v1) * tau) / tau ** 3
        K = max(1, int(np.ceil(tau / DT)))
        assert st["step"][p] == st["step"][q] + K
        hit, doubt = np.zeros(sc.N, bool), np.zeros(sc.N, bool)
        for k in range(1, K + 1):
            t = k * tau / K
            a, b = hsmc.halfspaces(x0[:3] + t * (v0 + t * (c2 + t * c3)), v0 + t * (2 * c2 + 3 * t * c3), boxes)
            dy = D[st["step"][q] + k].astype(np.float64)
            hit |= hsmc.violations(a, b, dy)
            doubt |= np.abs(hsmc.margins(a, b, dy)) < 1e-9
        want = bits[q] | hit
        same = (bits[p] == want) | doubt
        assert same.all(), (p, np.nonzero(~same)[0])
        assert st["pop"][p] == bits[p].sum()
        hits += int((want & ~bits[q]).sum())
    return len(order), hits


@pytest.mark.parametrize("N,n_obs,sigma", [(32, 0, 0.02), (32, 3, 0.03), (64, 64, 0.05), (128, 65, 0.05),
                                           (256, 20, 0.06), (128, 130, 0.08)])
def test_bits(N, n_obs, sigma):
    print_case("half batches", N=N, n_obs=n_obs, sigma=sigma)
    side = (0.1, 0.3) if n_obs <= 20 else (0.02, 0.08)
    sc = scenes.make_scene(dict(n=160, n_obs=n_obs, side=side, N=N, sigma=sigma, alpha=0.6, indoor=False),
                           41 + N + n_obs, M=256, S_max=160)
    pl = planner_for(sc, cp_model=1)
    pr = pl.scene_problem(sc, device=True)
    stores = []
    for mode in (1, 0):
        pl.set_explore_mode(mode)
        r = pl.plan(pr)
        stores.append((r, pl.plans()))
    for k in stores[0][1]:
        np.testing.assert_array_equal(stores[0][1][k], stores[1][1][k], err_msg=k)
    for k in ("simulated", "preprune", "inserted", "flagged", "sim_waypoints", "sim_box_tests"):
        assert stores[0][0][k] == stores[1][0][k], k
    n, hits = _check(stores[0][1], pl.graph(sc.n + 1), sc, pl.deviation(), 150)
    print("  plans", n, "of", len(stores[0][1]["head"]), "new hits", hits, flush=True)
    assert n > 20 and (hits > 0 or n_obs == 0)
    pl.close()
