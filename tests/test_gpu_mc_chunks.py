"""MC(p) at the edges of its split: 64 particles a workgroup (the last one
partly filled), chunks of 16 steps, boxes in one to four words of 64.  The
count equals the FP64 oracle's (a particle within rounding of a box's face has
a probability below 1e-10 here)."""

import numpy as np
import pytest

from oracle import dynamics, select as osel, steer as st
from paper_1607_06886_amd import _lib
from tests._gpu import CFG, print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,S,n_obs", [(1, 16, 1), (63, 1, 65), (64, 15, 1), (65, 16, 64), (257, 17, 65),
                                       (1000, 32, 256), (1000, 33, 3), (130, 48, 0)])
def test_count(M, S, n_obs):
    print_case("mc chunks", M=M, S=S, n_obs=n_obs)
    rng = np.random.default_rng(M + S)
    samples = np.array([[0.9, 0.5, 0.5, 0.0, 0.0, 0.0]], np.float32)
    x0 = np.array([0.1, 0.5, 0.5, 0, 0, 0], np.float32)
    V = np.concatenate([x0[None], samples]).astype(np.float64)
    tau, _ = st.steer(V[:1], V[1:], CFG.r_steer)
    dt = float(np.float32(float(tau[0]) / (S - 0.5) if S > 1 else float(tau[0]) * 1.5))
    # boxes beside the way, the first few within reach of the particles
    c = np.stack([rng.uniform(0.2, 0.8, n_obs), rng.choice([-1.0, 1.0], n_obs) * rng.uniform(0.01, 0.35, n_obs),
                  rng.uniform(-0.3, 0.3, n_obs)], 1)
    c[:, 1:] += 0.5
    h = rng.uniform(0.002, 0.008, (n_obs, 3))
    if n_obs:
        c[0], h[0] = [0.5, 0.56, 0.5], [0.2, 0.045, 0.2]
    boxes = np.concatenate([c - h, c + h], 1).astype(np.float32)
    noise = rng.standard_normal((64, 6, 32), dtype=np.float32)
    noise_mc = rng.standard_normal((64, 6, M), dtype=np.float32)
    sigma = 0.03
    pl = _lib.Planner(n_particles=32, max_nodes=2, max_obstacles=max(n_obs, 1), max_steps=64, mc_particles=M,
                      cap_plans=1024, cap_pairs=1024, cap_edges=1024, dt=dt, r_conn=min(1.0, 30 * dt))
    pl.setup(pl.problem(samples, boxes, x0, [0.85, 0.45, 0.45, 0.95, 0.55, 0.55], 0.05, sigma, noise, noise_mc))
    got = pl.mc_path([0, 1])
    pl.close()
    A_cl, L, _ = dynamics.closed_loop(dt, float(np.float32(sigma)), CFG.q_pos, CFG.q_vel, CFG.r_track)
    W = osel.plan_waypoints(V, (0, 1), CFG.r_steer, dt)
    assert len(W) == S + 1
    want = osel.mc_count_waypoints(W, boxes, A_cl, L, noise_mc)
    print("  colliding", got, "of", M, flush=True)
    assert got == want
    assert n_obs != 3 or 0 < want < M
