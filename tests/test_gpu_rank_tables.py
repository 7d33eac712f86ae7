"""The box model's particle bits, found by rank (rank_tables.hpp), against a
test of every particle: each plan's bits are its parent's and those of the
particles inside some box at some waypoint of its edge, from the library's own
deviation table.  Cases at the edges of the tables: every particle count, box
sets of one to four 64-bit words, all deviations equal (sigma = 0), particles
that are NaN or infinite from some step on, and teams of one workgroup (many
passes of pairs each) beside the whole device (one short pass each).

Positions are of order 1, so the nominal points of the two sides differ by
some 1e-15; a particle within 1e-12 of a face (an FP32 deviation lies there by
chance once in about 1e8 decisions) is left out."""

import numpy as np
import pytest

from paper_1607_06886_amd import _lib, scenes
from tests._gpu import planner_for, print_case

pytestmark = pytest.mark.gpu

SLACK = 1e-12
DT = float(np.float32(0.05))


def _scene(N, n_obs, sigma, special, seed):
    side = (0.1, 0.3) if n_obs <= 20 else (0.02, 0.09)
    sc = scenes.make_scene(dict(n=260, n_obs=n_obs, side=side, N=N, sigma=sigma, alpha=0.2,
                                indoor=False), seed, M=256, S_max=160)
    if special == "nan":
        sc.noise[3, 0, 5] = np.nan      # particle 5 on axis 0 from step 4 on
        sc.noise[9, 4, N - 1] = np.nan
    elif special == "inf":
        sc.noise[3, 0, 5] = np.inf
        sc.noise[4, 2, 7] = -np.inf
    return sc


def _edge_hits(x0, x1, tau, s_p, D, boxes):
    """Hits and doubtful bits of an edge's waypoints, over all particles."""
    K = max(1, int(np.ceil(tau / DT)))
    x0, x1 = x0.astype(np.float64), x1.astype(np.float64)
    P, v0, v1 = x1[:3] - x0[:3], x0[3:], x1[3:]
    c2 = (3 * P - (2 * v0 + v1) * tau) / tau ** 2
    c3 = (-2 * P + (v0 + v1) * tau) / tau ** 3
    N = D.shape[2]
    hit, doubt = np.zeros(N, bool), np.zeros(N, bool)
    for k in range(1, K + 1):
        t = k * tau / K
        y = (x0[:3] + t * (v0 + t * (c2 + t * c3)))[:, None] + D[s_p + k].astype(np.float64)
        for b in boxes.astype(np.float64):
            d = np.minimum(y - b[:3, None], b[3:, None] - y)
            d = np.where(np.isnan(d).any(0), -np.inf, d.min(0))
            hit |= d >= 0.0
            doubt |= np.abs(d) < SLACK
    return K, hit, doubt


def _check_store(pl_plans, graph, sc, D):
    X = np.concatenate([sc.x_init[None], sc.samples])
    bits = np.unpackbits(pl_plans["mask"].view(np.uint8), axis=1, bitorder="little").astype(bool)
    n_checked = n_hits = 0
    for p in range(1, len(pl_plans["head"])):
        q = pl_plans["parent"][p]
        e = pl_plans["edge"][p]
        K, hit, doubt = _edge_hits(X[pl_plans["head"][q]], X[pl_plans["head"][p]], graph["tau"][e],
                                   pl_plans["step"][q], D, sc.obstacles)
        assert pl_plans["step"][p] == pl_plans["step"][q] + K
        want = bits[q] | hit
        same = (bits[p] == want) | doubt
        assert same.all(), (p, np.nonzero(~same)[0])
        assert pl_plans["pop"][p] == bits[p].sum()
        n_checked += 1
        n_hits += int((want & ~bits[q]).sum())
    return n_checked, n_hits


CASES = [(32, 3, 0.02, ""), (64, 64, 0.02, ""), (64, 65, 0.03, ""), (128, 129, 0.02, ""),
         (256, 256, 0.02, ""), (256, 20, 0.05, ""), (128, 20, 0.0, ""), (32, 20, 0.03, "nan"),
         (256, 20, 0.03, "nan"), (128, 20, 0.03, "inf"), (64, 0, 0.02, "")]


@pytest.mark.parametrize("N,n_obs,sigma,special", CASES)
def test_bits_by_rank_equal_bits_by_particle(N, n_obs, sigma, special):
    print_case("bits by rank", N=N, n_obs=n_obs, sigma=sigma, special=special)
    sc = _scene(N, n_obs, sigma, special, 31 + N + n_obs)
    pl = planner_for(sc)
    pr = pl.scene_problem(sc, device=True)
    stores = []
    for mode in (1, 0):
        pl.set_explore_mode(mode)
        r = pl.plan(pr)
        stores.append((r, pl.plans()))
    for k in stores[0][1]:
        np.testing.assert_array_equal(stores[0][1][k], stores[1][1][k], err_msg=k)
    n_checked, n_hits = _check_store(stores[0][1], pl.graph(sc.n + 1), sc, pl.deviation())
    print("  plans", n_checked, "new hits", n_hits, flush=True)
    assert n_checked > 50
    assert n_hits > 0 or n_obs == 0 or sigma == 0.0
    pl.close()


@pytest.mark.parametrize("team_scale", [0, 64])
def test_batched_teams_equal_the_single_query(team_scale):
    """One workgroup per query takes its pairs in many passes, a large team in
    one short pass each; both equal pump_plan's result."""
    print_case("bits by rank, batched", team_scale=team_scale)
    import torch
    cases = [(32, 3, 0.02, ""), (64, 65, 0.03, ""), (256, 20, 0.05, "nan")]
    scs = [_scene(*c, 31 + c[0] + c[1]) for c in cases]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    b = _lib.Batch(len(scs), n_particles=256, max_nodes=261, max_obstacles=65, max_steps=160,
                   mc_particles=256, cap_plans=1 << 16, cap_pairs=1 << 18, cap_edges=1 << 18)
    got = b.plan([(dev(s.samples), dev(s.obstacles), s.x_init, s.goal, s.alpha, s.sigma,
                   dev(s.noise), dev(s.noise_mc)) for s in scs], dict(team_scale=team_scale))
    b.close()
    for sc, r in zip(scs, got):
        pl = planner_for(sc)
        ref = pl.plan(pl.scene_problem(sc, device=True))
        pl.close()
        for k in ("status", "best_plan", "best_cost", "best_mc_count", "partial_plans", "simulated",
                  "preprune", "inserted", "flagged", "sim_waypoints", "sim_box_tests", "n_plans"):
            assert r[k] == ref[k], k
