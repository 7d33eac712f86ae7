"""Paths read back from the device: every plan of a store, ids outside it, and
the slots of queries that have no plans (refused inputs)."""

import dataclasses

import numpy as np
import pytest

from paper_1607_06886_amd import _lib
from tests._gpu import gpu_plans, planner_for, print_case, scene

pytestmark = pytest.mark.gpu


def test_every_plan_and_ids_outside_the_store():
    print_case("paths of a store")
    sc = scene("cfg1", 1)
    pl = planner_for(sc)
    pl.plan(pl.scene_problem(sc, device=True))
    st = gpu_plans(pl)
    n = len(st["head"])
    assert n > 20
    for p in range(n):
        assert pl.path(p) == st["paths"][p], p
    for p in (-1, n, n + 1, 2**31 - 1):
        with pytest.raises(_lib.PumpError):
            pl.path(p)
    pl.close()


def test_refused_query_has_no_paths():
    print_case("paths of refused queries")
    import torch
    good = scene("cfg1", 1)
    bad = dataclasses.replace(good, samples=good.samples + np.float32(20.0))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    b = _lib.Batch(3, n_particles=32, max_nodes=good.n + 1, max_obstacles=good.n_obs,
                   max_steps=good.S_max, mc_particles=good.M, cap_plans=1 << 16, cap_pairs=1 << 18,
                   cap_edges=1 << 18)
    res = b.plan([(dev(s.samples), dev(s.obstacles), s.x_init, s.goal, s.alpha, s.sigma, dev(s.noise),
                   dev(s.noise_mc)) for s in (bad, good, bad)], raise_on_error=False)
    assert [r["status"] < 0 for r in res] == [True, False, True]
    for i in (0, 2):
        for p in (0, 1, (1 << 16) - 1, 2**31 - 1):
            with pytest.raises(_lib.PumpError):
                b.path(i, p)
    assert b.path(1, 0) == (0,)
    assert b.path(1, res[1]["best_plan"])[0] == 0
    b.close()
