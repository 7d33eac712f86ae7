"""Clouds as wide as the boxes are apart: records tested by particle instead of by
rank, in the workgroup that found them and, once half of a round's are wide,
through the round's queue.  Each plan's bits against a test of every particle
(test_gpu_rank_tables), the same plan store whichever way the rounds run, and the
counts of flagged decisions against the oracle's."""

import numpy as np
import pytest

from paper_1607_06886_amd import _lib, scenes
from tests._gpu import CFG, opump, planner_for, print_case
from tests.test_gpu_rank_tables import _edge_hits

pytestmark = pytest.mark.gpu

SAME = ("status", "partial_plans", "simulated", "preprune", "inserted", "survivors", "dropped_steps", "flagged",
        "rounds", "n_plans", "best_plan", "best_cost", "best_mc_count", "sim_waypoints", "sim_box_tests")

# (a chunk may resolve a pair by the chunks before it)
CHUNKS_SAME = [k for k in SAME if k not in ("simulated", "preprune", "inserted", "flagged", "sim_waypoints",
                                            "sim_box_tests")]


def _scene(n, N, n_obs, sigma, seed, side=(0.02, 0.09)):
    return scenes.make_scene(dict(n=n, n_obs=n_obs, side=side, N=N, sigma=sigma, alpha=0.4, indoor=False),
                             seed, M=256, S_max=160)


def _check_plans(st, graph, sc, D, limit):
    """Bits of up to `limit` plans against their parents' and a test of every
    particle at every waypoint of their last edge."""
    X = np.concatenate([sc.x_init[None], sc.samples])
    bits = np.unpackbits(st["mask"].view(np.uint8), axis=1, bitorder="little").astype(bool)
    hits = 0
    order = np.random.default_rng(0).permutation(np.arange(1, len(st["head"])))[:limit]
    for p in order:
        q, e = st["parent"][p], st["edge"][p]
        _, hit, doubt = _edge_hits(X[st["head"][q]], X[st["head"][p]], graph["tau"][e], st["step"][q], D,
                                   sc.obstacles)
        want = bits[q] | hit
        assert ((bits[p] == want) | doubt).all(), p
        assert st["pop"][p] == bits[p].sum()
        hits += int((want & ~bits[q]).sum())
    return len(order), hits


# box sets of one, two and four 64-bit words; particles below, at and above a wave
@pytest.mark.parametrize("N,n_obs,sigma", [(32, 64, 0.18), (64, 64, 0.15), (128, 65, 0.12), (256, 40, 0.12),
                                           (256, 200, 0.09)])
def test_bits_and_stores(N, n_obs, sigma):
    print_case("wide clouds", N=N, n_obs=n_obs, sigma=sigma)
    sc = _scene(400, N, n_obs, sigma, 60 + N + n_obs)
    ref = None
    for mode, caps in ((0, {}), (1, {}), (0, dict(cap_pairs=2048))):
        pl = planner_for(sc, **caps)
        pl.set_explore_mode(mode)
        r = pl.plan(pl.scene_problem(sc, device=True))
        st = pl.plans()
        if ref is None:
            ref = r, st
            print("  pairs", r["partial_plans"], "rounds", r["rounds"], "waypoints", r["sim_waypoints"],
                  "box tests", r["sim_box_tests"], "flagged", r["flagged"], flush=True)
            # (rounds of some hundreds of wide records, so the queue is on in some)
            assert r["rounds"] >= 3 and r["simulated"] >= 400 * r["rounds"]
            assert r["sim_box_tests"] >= 3 * r["sim_waypoints"]
            n, hits = _check_plans(st, pl.graph(sc.n + 1), sc, pl.deviation(), 400)
            print("  plans", n, "new hits", hits, flush=True)
            assert n > 50 and hits > 0
        elif caps:
            assert pl.chunked_rounds() > 0
        for k in SAME if not caps else CHUNKS_SAME:
            assert r[k] == ref[0][k], (mode, caps, k)
        for k in st:
            np.testing.assert_array_equal(st[k], ref[1][k], err_msg=f"{mode} {caps} {k}")
        pl.close()


@pytest.mark.parametrize("N,tuning", [(64, None), (256, dict(team_scale=0)), (256, dict(team_scale=64))])
def test_batched_teams(N, tuning):
    print_case("wide clouds, batched", N=N, tuning=tuning)
    import torch
    scs = [_scene(320, N, 40, 0.12, 60 + N + 40), _scene(150, N, 20, 0.15, 5)]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    b = _lib.Batch(len(scs), n_particles=N, max_nodes=321, max_obstacles=64, max_steps=160, mc_particles=256,
                   cap_plans=1 << 18, cap_pairs=1 << 20, cap_edges=1 << 18)
    got = b.plan([(dev(s.samples), dev(s.obstacles), s.x_init, s.goal, s.alpha, s.sigma, dev(s.noise),
                   dev(s.noise_mc)) for s in scs], tuning)
    b.close()
    for sc, r in zip(scs, got):
        pl = planner_for(sc)
        ref = pl.plan(pl.scene_problem(sc, device=True))
        pl.close()
        for k in SAME:
            assert r[k] == ref[k], k


def test_flagged_counts_equal_the_oracle():
    """Without early resolution the library tests exactly the pairs the oracle
    extends, so the flagged decisions of those below the cutoff agree."""
    print_case("wide clouds, flagged")
    sc = _scene(110, 256, 24, 0.12, 3)
    ref = opump.run(sc, CFG)
    want = ref["stats"]["flagged_below_cut"]
    assert want > 0
    for mode in (0, 1):
        pl = planner_for(sc, preprune=0)
        pl.set_explore_mode(mode)
        r = pl.plan(pl.scene_problem(sc, device=True))
        pl.close()
        assert r["partial_plans"] == ref["stats"]["partial_plans"]
        assert r["sim_box_tests"] >= 2.5 * r["sim_waypoints"]
        assert r["flagged"] == want


@pytest.mark.parametrize("N,special", [(32, np.nan), (256, np.nan), (64, np.inf), (256, -np.inf)])
def test_positions_that_are_no_numbers(N, special):
    """A particle without a position on some axis is in no box, whichever way its
    record is tested (by rank: test_gpu_rank_tables)."""
    print_case("wide clouds, not finite", N=N, special=special)
    sc = _scene(400, N, 40, 0.15, 60 + N)
    for j, (step, row) in enumerate([(1, 0), (2, 2), (4, 4), (1, 1)]):   # particles 5, 12, 19, 26
        sc.noise[step, row, 5 + 7 * j] = special
    ref = None
    for mode in (0, 1):
        pl = planner_for(sc)
        pl.set_explore_mode(mode)
        r = pl.plan(pl.scene_problem(sc, device=True))
        st, D = pl.plans(), pl.deviation()
        if ref is None:
            assert not np.isfinite(D[6:]).all(axis=(0, 1))[[5, 12, 19, 26]].any()
            with np.errstate(invalid="ignore"):
                n, hits = _check_plans(st, pl.graph(sc.n + 1), sc, D, 400)
            print("  plans", n, "new hits", hits, "box tests", r["sim_box_tests"], "waypoints", r["sim_waypoints"],
                  flush=True)
            assert n > 50 and hits > 0 and r["sim_box_tests"] >= 3 * r["sim_waypoints"]
            ref = st
        for k in st:
            np.testing.assert_array_equal(st[k], ref[k], err_msg=f"{mode} {k}")
        pl.close()


def test_flagged_counts_of_half_waves():
    """(32 particles: each half of a wave tests every other box.)"""
    print_case("wide clouds, flagged, 32 particles")
    sc = _scene(220, 32, 25, 0.12, 3)
    sc.obstacles[:, 2] = np.float32(0.0)     # boxes from the floor up: more decisions near a face
    ref = opump.run(sc, CFG)
    for mode in (0, 1):
        pl = planner_for(sc, preprune=0)
        pl.set_explore_mode(mode)
        r = pl.plan(pl.scene_problem(sc, device=True))
        pl.close()
        print("  flagged", r["flagged"], ref["stats"]["flagged_below_cut"], "box tests", r["sim_box_tests"], "waypoints",
              r["sim_waypoints"], flush=True)
        assert r["partial_plans"] == ref["stats"]["partial_plans"]
        assert r["sim_box_tests"] >= 2 * r["sim_waypoints"]
        assert r["flagged"] == ref["stats"]["flagged_below_cut"]
    assert ref["stats"]["flagged_below_cut"] > 0
