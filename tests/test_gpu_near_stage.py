"""BuildGraph's near stage at the edges of its split: workgroups of 4 rows (and
a last one of fewer), chunks of 1024 targets, a radius within which nearly
every pair is kept (the list is steered between chunks) and one that keeps
next to none, repeated and unreachable states.  Adjacency, tau* and c* of the
first and last rows against the FP64 oracle (relative 1e-9, as the parity
tests of whole graphs)."""

import numpy as np
import pytest

from oracle import graph as ogr
from paper_1607_06886_amd import scenes
from tests._gpu import CFG, planner_for, print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r_conn", [(1, 1.0), (2, 1.0), (3, 1.0), (4, 1.0), (66, 1.0), (1022, 1.0), (1023, 1.0),
                                      (1024, 1.0), (2051, 0.3), (1500, 4.0)])
def test_rows(n, r_conn):
    print_case("near stage", n=n, r_conn=r_conn)
    sc = scenes.make_scene(dict(n=max(n, 8), n_obs=2, side=(0.1, 0.2), N=32, sigma=0.02, alpha=0.1,
                                indoor=False), 17, M=256, S_max=96)
    sc.samples = np.ascontiguousarray(sc.samples[-n:])
    if n > 60:
        sc.samples[20] = sc.samples[21]                  # the same state twice
        sc.samples[30, 3:] = 40.0                        # hard to reach and to leave
        sc.samples[31, 3:] = 0.0
    pl = planner_for(sc, max_nodes=n + 1, r_conn=r_conn, dt=0.2)   # (4 is more than 64 steps of 0.05)
    pl.setup(pl.scene_problem(sc))
    g = pl.graph(n + 1)
    pl.close()
    V = np.concatenate([sc.x_init[None], sc.samples]).astype(np.float64)
    valid = ~ogr.points_in_boxes(V[:, :3], sc.obstacles)
    np.testing.assert_array_equal(g["valid"], valid)
    rows = sorted({*range(0, min(n + 1, 6)), *range(max(0, n - 5), n + 1), *([21, 22, 31, 32] if n > 60 else [])})
    src, dst, tau, cost = ogr.graph_rows(V, valid, sc.obstacles, float(np.float32(r_conn)), CFG.r_steer, rows)
    order = np.lexsort((dst, src))
    src, dst, tau, cost = src[order], dst[order], tau[order], cost[order]
    for v in rows:
        lo, hi = g["row_ptr"][v], g["row_ptr"][v + 1]
        np.testing.assert_array_equal(g["col"][lo:hi], dst[src == v], err_msg=str(v))
        np.testing.assert_allclose(g["tau"][lo:hi], tau[src == v], rtol=1e-9)
        np.testing.assert_allclose(g["cost"][lo:hi], cost[src == v], rtol=1e-9)
    print("  edges", len(g["col"]), "in the rows", len(dst), flush=True)
