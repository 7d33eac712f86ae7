"""The half-space model at nodes at rest.  The nominal velocity at the last
waypoint of such an edge is zero but for the rounding of its cubic's slope, and
its direction, so the plane eq. (7) leaves, is that rounding's: the slope is
one chain of fused multiply-adds, c1 + t (2 c2 + (3 t) c3), in every build.

The reference evaluates that chain exactly and rounds each step once."""

from fractions import Fraction

import numpy as np
import pytest

from oracle import hsmc
from paper_1607_06886_amd import scenes
from tests._gpu import planner_for, print_case, unpack_mask

pytestmark = pytest.mark.gpu


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _waypoint(x0, x1, tau, k, K):
    it = 1.0 / tau
    it2 = it * it
    it3 = it2 * it
    t = (k * tau) / K
    y, v = [], []
    for ax in range(3):
        p0 = float(x0[ax])
        P = float(x1[ax]) - p0
        c2, c3 = (3.0 * P) * it2, (-2.0 * P) * it3      # (no velocity at either end)
        y.append(_fma(t, _fma(t, _fma(t, c3, c2), 0.0), p0))
        v.append(_fma(t, _fma(3.0 * t, c3, 2.0 * c2), 0.0))
    return y, v


def _planes(y, v, boxes):
    vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2]
    for d in hsmc.local_region(y, boxes).tolist():
        f = ((d[0] * v[0] + d[1] * v[1]) + d[2] * v[2]) / vv if vv > 0.0 else 0.0
        a = [d[i] - f * v[i] for i in range(3)]
        yield np.array(a), (a[0] * a[0] + a[1] * a[1]) + a[2] * a[2]


@pytest.mark.parametrize("N", [32, 128])
def test_planes_at_rest(N):
    print_case("half-space, nodes at rest", N=N)
    sc = scenes.make_scene(dict(n=200, n_obs=6, side=(0.1, 0.25), N=N, sigma=0.05, alpha=0.6, indoor=False),
                           5, M=256, S_max=128)
    sc.samples[:, 3:] = 0.0
    sc.x_init[3:] = 0.0
    pl = planner_for(sc, cp_model=1)
    pr = pl.scene_problem(sc, device=True)
    for mode in (0, 1):
        pl.set_explore_mode(mode)
        pl.plan(pr)
        st, g, D = pl.plans(), pl.graph(sc.n + 1), pl.deviation().astype(np.float64)
        X = np.concatenate([sc.x_init[None], sc.samples]).astype(np.float32)
        pick = np.arange(1, len(st["head"]))
        pick = pick[np.linspace(0, len(pick) - 1, min(len(pick), 120)).astype(int)]
        sure = wrong = hits = 0
        for q in pick:
            p, e = int(st["parent"][q]), int(st["edge"][q])
            s_p, K = int(st["step"][p]), int(st["step"][q] - st["step"][p])
            hit, close = np.zeros(N, bool), np.zeros(N, bool)
            for k in range(1, K + 1):
                dy = D[s_p + k]
                y, v = _waypoint(X[st["head"][p]], X[st["head"][q]], float(g["tau"][e]), k, K)
                for a, b in _planes(y, v, sc.obstacles):
                    over = a @ dy - b
                    hit |= over > 0.0
                    # g's rounding: some four units of 2^-53 of |a| |dy| and of b
                    close |= np.abs(over) <= 1e-14 * (np.linalg.norm(a) * np.linalg.norm(dy, axis=0) + b)
            par = unpack_mask(st["mask"][p], N)
            got = unpack_mask(st["mask"][q], N)
            ok = par | ~close
            sure += int(ok.sum())
            hits += int((hit & ~par).sum())
            wrong += int(((par | hit) != got)[ok].sum())
        print("  mode", mode, "plans", len(pick), "of", len(st["head"]), "sure", sure, "hits", hits, "wrong", wrong,
              flush=True)
        assert sure > 0.9 * N * len(pick) and hits > 0
        assert wrong == 0
    pl.close()
