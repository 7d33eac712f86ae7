"""Performance cases: what programs written against this package have it do.

Every case is one call sequence of a user's program through the package's
public entry points (`Planner`, `Roadmap`, `Batch`, `MLP`, `sample_halton`):

  query   one planning query: `Planner.plan`, then the certified plan's path
          (or, when no plan is certified, the front and its Monte Carlo
          counts).  Maps: random boxes, the indoor room grid, or random boxes
          with half of the samples crowded along the start-goal corridor, as
          a learned proposal places them.  Options in use: the half-space
          exploration model, LQG tracking, the final smoothing, Halton
          samples drawn per query, a cached roadmap.
  batch   many queries in one `Batch.plan`, then each certified plan's path.
  train   training steps of the proposal network, then its parameters.
  forward / sample   the network's outputs for a batch of conditions; draws
          from its mixture for one map, from the map's arrays on.

Inputs live on the device, as they do in the benchmark and in the training
driver.  Sizes and distributions are those of the package's own workloads
(3 boxes / 500 samples / 32 particles up to the indoor map with 20,000
samples / 256 particles, and batches with 1000 to 8000 samples a query).
"""

import math
import os

import numpy as np
import torch

import paper_1607_06886_amd
from paper_1607_06886_amd import _lib, scenes

S_MAX = 512
MC = 10_000
NET_IN, NET_OUT, COMPONENTS = 396, 208, 16
LAYERS = [(396, 256), (256, 256), (256, 256), (256, 256), (256, 208)]
BETA1, BETA2, EPS = 0.9, 0.999, 1e-8
LEARNING_RATE = 1e-4   # a trained network taken further on other maps
ADAM_T0 = 500          # step counter of the checkpoint that training resumes
ADAM_M2 = 1e-2         # its second moments, about the gradients' squares
WEIGHTS = os.path.join(os.path.dirname(paper_1607_06886_amd.__file__), "weights",
                       "proposal_params.npy")


def _query(name, kind, n, N, n_obs, alpha, **opt):
    c = dict(name=name, what="query", map=kind, n=n, N=N, n_obs=n_obs, alpha=alpha, hsmc=False,
             lqg=False, smooth=False, halton=False, roadmap=False)
    c.update(opt)
    return c


def listed():
    return [
        # the smallest query: a few boxes, few particles; latency and launches
        _query("boxes_500", "boxes", 500, 32, 3, 0.05),
        # every option of an on-line planner at an odd size: Halton samples
        # per query, LQG tracking, the final smoothing
        _query("boxes_2333_halton_lqg_smooth", "boxes", 2333, 64, 37, 0.05, lqg=True, smooth=True,
               halton=True),
        # the ordinary query (the paper's particle count)
        _query("boxes_4000", "boxes", 4000, 128, 20, 0.01),
        # the same with the paper's own exploration model
        _query("boxes_4000_halfspace", "boxes", 4000, 128, 20, 0.01, hsmc=True),
        # half learned, half uniform samples at the evaluation size
        _query("corridor_8000", "corridor", 8000, 256, 33, 0.01),
        # offline graph, on-line obstacles: indoor map over a cached roadmap
        _query("indoor_11111_roadmap", "indoor", 11111, 128, 60, 0.01, roadmap=True),
        # the largest single query: the benchmark's workload
        _query("indoor_20000", "indoor", 20000, 256, 60, 0.01),
        # a serving batch of uneven queries
        dict(name="batch_64_uneven", what="batch", q=64, n_lo=1000, n_hi=8000, mixed=True),
        # a batch of training maps (even sizes, shared particle noise)
        dict(name="batch_96_training_maps", what="batch", q=96, n_lo=2000, n_hi=2000, mixed=False),
        # training: eight minibatches of the training driver's size
        dict(name="train_2048", what="train", B=2048, steps=8),
        # inference over many maps, an odd batch
        dict(name="forward_4999", what="forward", B=4999),
        # the proposal's draws of one query of 8000 samples: the smallest call
        dict(name="sample_4000", what="sample", n=4000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["boxes"] * 4 + ["options"] * 2 + ["corridor", "indoor", "indoor", "batch",
                                                         "train", "forward", "sample"])
    alpha = rng.choice([0.01, 0.05])
    if kind == "boxes":
        return _drawn(_query("", "boxes", _log_int(rng, 300, 8000), rng.choice([32, 64, 128, 256]),
                             rng.randint(3, 60), alpha, roadmap=rng.random() < 0.25))
    if kind == "options":
        hsmc = rng.random() < 0.5
        return _drawn(_query("", "boxes", _log_int(rng, 500, 4000), rng.choice([64, 128]),
                             rng.randint(5, 30), 0.01 if hsmc else alpha, hsmc=hsmc,
                             lqg=rng.random() < 0.5, smooth=rng.random() < 0.7,
                             halton=rng.random() < 0.5))
    if kind == "corridor":
        return _drawn(_query("", "corridor", _log_int(rng, 1000, 8000), rng.choice([128, 256]),
                             rng.randint(5, 60), 0.01))
    if kind == "indoor":
        return _drawn(_query("", "indoor", _log_int(rng, 2000, 20000), rng.choice([64, 128, 256]),
                             60, 0.01, roadmap=rng.random() < 0.4))
    if kind == "batch":
        lo = _log_int(rng, 700, 2500)
        return dict(what="batch", q=rng.randint(9, 48), n_lo=lo, n_hi=rng.randint(lo, 6000),
                    mixed=True)
    if kind == "train":
        return dict(what="train", B=_log_int(rng, 64, 2048), steps=8)
    if kind == "forward":
        return dict(what="forward", B=_log_int(rng, 1, 8192))
    return dict(what="sample", n=_log_int(rng, 100, 8000))


def _drawn(c):
    c.pop("name")
    return c


# --------------------------------------------------------------------------
# planning queries
# --------------------------------------------------------------------------
def _rng(seed, stream):
    return np.random.default_rng([int(seed), 7000 + stream])


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def _normals(shape, seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + stream)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _map(kind, n_obs, rng):
    """(x_init, goal box, boxes) of one query."""
    if kind == "indoor":
        c = np.asarray(scenes.INDOOR_GOAL_CENTRE)
        goal = np.concatenate([c - scenes.INDOOR_GOAL_HALF, c + scenes.INDOOR_GOAL_HALF])
        return (np.asarray(scenes.INDOOR_X_INIT, np.float32), goal.astype(np.float32),
                scenes.indoor_boxes(rng))
    x_init = np.asarray(scenes.X_INIT, np.float32)
    goal = np.asarray(scenes.GOAL_BOX, np.float32)
    side = (0.1, 0.3) if n_obs <= 4 else (0.05, 0.25)
    return x_init, goal, scenes.random_boxes(rng, n_obs, side, x_init, goal)


def _samples(kind, n, boxes, x_init, goal, rng):
    n_goal = max(1, int(math.ceil(0.01 * n)))
    if kind != "corridor":
        return scenes.free_samples(rng, n, boxes, goal, n_goal)
    # half of the samples in 16 clusters along the line from start to goal,
    # moving towards the goal (some lie in obstacles and are dropped), half
    # uniform
    half = n // 2
    c = 0.5 * (goal[:3] + goal[3:])
    t = rng.integers(0, COMPONENTS, half)[:, None] / (COMPONENTS - 1.0)
    pos = x_init[:3] + t * (c - x_init[:3]) + 0.08 * rng.standard_normal((half, 3))
    vel = 0.25 * (c - x_init[:3]) + 0.15 * rng.standard_normal((half, 3))
    crowd = np.concatenate([np.clip(pos, 0.0, 1.0),
                            np.clip(vel, -scenes.VEL_HALF, scenes.VEL_HALF)], axis=1)
    rest = scenes.free_samples(rng, n - half, boxes, goal, n_goal)
    return np.concatenate([crowd.astype(np.float32), rest])


def _prepare_query(case, seed):
    n, N = case["n"], case["N"]
    rng = _rng(seed, 0)
    x_init, goal, boxes = _map(case["map"], case["n_obs"], rng)
    big = n > 8000
    cfg = dict(n_particles=N, max_nodes=n + 1, max_obstacles=len(boxes), max_steps=S_MAX,
               mc_particles=MC, cap_plans=1 << 22 if big else 1 << 21,
               cap_pairs=1 << 25 if big else 1 << 24, cap_edges=1 << 25,
               cp_model=int(case["hsmc"]), estimator=int(case["lqg"]), smooth=int(case["smooth"]))
    st = dict(pl=_lib.Planner(**cfg), boxes=_dev(boxes), x_init=x_init, goal=goal,
              alpha=case["alpha"], sigma=0.01 if len(boxes) <= 4 else 0.02,
              noise=_normals((S_MAX, 6, N), seed, 1), noise_mc=_normals((S_MAX, 6, MC), seed, 2),
              meas=())
    if case["lqg"]:
        st["meas"] = (0.01, _normals((S_MAX, 3, N), seed, 3), _normals((S_MAX, 3, MC), seed, 4))
    if case["halton"]:
        st["halton"] = (n, max(1, n // 100), 1 + int(rng.integers(0, 1 << 20)))
    else:
        st["samples"] = _dev(_samples(case["map"], n, boxes, x_init, goal, rng))
    if case["roadmap"]:
        st["rm"] = _lib.Roadmap(st["samples"], max_nodes=n + 1, cap_edges=1 << 25)
        st["pl"].set_roadmap(st["rm"])
    return st


STATE_LO = [0.0, 0.0, 0.0, -scenes.VEL_HALF, -scenes.VEL_HALF, -scenes.VEL_HALF]
STATE_HI = [1.0, 1.0, 1.0, scenes.VEL_HALF, scenes.VEL_HALF, scenes.VEL_HALF]


def _outcome(r):
    """A result record without its times."""
    return {k: v for k, v in r.items() if not k.startswith("ms_")}


def _run_query(st):
    pl, out = st["pl"], {}
    samples = st.get("samples")
    if samples is None:
        n, n_goal, start = st["halton"]
        samples = _lib.sample_halton(n, STATE_LO, STATE_HI, st["goal"], n_goal, start)
        out["samples"] = samples
    pr = pl.problem(samples, st["boxes"], st["x_init"], st["goal"], st["alpha"], st["sigma"],
                    st["noise"], st["noise_mc"], *st["meas"])
    r = pl.plan(pr)
    out["result"] = _outcome(r)
    # node sequence of the plan, or plan ids and counts of the front (-1 past
    # their ends)
    found = np.full((2, S_MAX + 1), -1, np.int64)
    if r["status"] == 0:
        path = pl.path(r["best_plan"])
        found[0, :len(path)] = path
    else:
        for row, v in zip(found, pl.front()):
            row[:len(v)] = v
    out["found"] = found
    return out


def _exact_query(case, seed):
    # the drawn Halton points; the plan itself has no value without a planner
    if not case["halton"]:
        return None
    rng = _rng(seed, 0)
    _, goal, _ = _map(case["map"], case["n_obs"], rng)
    n, n_goal = case["n"], max(1, case["n"] // 100)
    start = 1 + int(rng.integers(0, 1 << 20))
    lo, hi = np.tile(STATE_LO, (n, 1)), np.tile(STATE_HI, (n, 1))
    lo[n - n_goal:, :3], hi[n - n_goal:, :3] = goal[:3], goal[3:]
    phi = np.zeros((n, 6))
    for d, b in enumerate((2, 3, 5, 7, 11, 13)):
        i, f = np.arange(start, start + n), 1.0 / b
        while i.any():
            phi[:, d] += f * (i % b)
            i, f = i // b, f / b
    return {"samples": lo + (hi - lo) * phi}


# --------------------------------------------------------------------------
# batches
# --------------------------------------------------------------------------
def _prepare_batch(case, seed):
    q, rng = case["q"], _rng(seed, 10)
    steps, mc = (S_MAX, MC) if case["mixed"] else (256, 2000)
    shared = None if case["mixed"] else (_normals((steps, 6, 128), seed, 1),
                                         _normals((steps, 6, mc), seed, 2))
    queries, ns = [], []
    for i in range(q):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        if case["mixed"]:
            N, alpha = int(rng.choice([64, 128, 256])), float(rng.choice([0.01, 0.05]))
            x_init, goal, boxes = _map("boxes", int(rng.integers(5, 61)), rng)
            noise = (_normals((steps, 6, N), seed, 100 + 2 * i),
                     _normals((steps, 6, mc), seed, 101 + 2 * i))
        else:
            N, alpha, noise = 128, 0.01, shared
            x_init, goal, boxes = scenes.random_map(("boxes", "indoor")[i % 2],
                                                    1000 * int(seed) + i)
        samples = scenes.free_samples(rng, n, boxes, goal, max(1, int(math.ceil(0.01 * n))))
        queries.append((_dev(samples), _dev(boxes), x_init, goal, alpha, 0.02) + noise)
        ns.append(n)
    b = _lib.Batch(q, n_particles=256 if case["mixed"] else 128, max_nodes=max(ns) + 1,
                   max_obstacles=64, max_steps=steps, mc_particles=mc, cap_plans=1 << 20,
                   cap_pairs=1 << 21, cap_edges=1 << 22)
    return dict(b=b, queries=queries)


def _run_batch(st):
    b = st["b"]
    res = b.plan(st["queries"], raise_on_error=False)
    out = {k: np.asarray([r[k] for r in res]) for k in res[0] if not k.startswith("ms_")}
    paths = np.full((len(res), b.cfg.max_steps + 1), -1, np.int64)   # (-1 past a path's end)
    for i, r in enumerate(res):
        if r["status"] == 0:
            path = b.path(i, r["best_plan"])
            paths[i, :len(path)] = path
    out["paths"] = paths
    return out


# --------------------------------------------------------------------------
# the proposal network
# --------------------------------------------------------------------------
def _params():
    return np.load(WEIGHTS, allow_pickle=False)


def _boxes_arrays(B, rng):
    """x_init [B, 6], goals [B, 6], boxes [B, 64, 6] and box counts of B maps."""
    x0 = np.zeros((B, 6), np.float32)
    x0[:, :3] = rng.uniform(0.05, 0.95, (B, 3))
    c = rng.uniform(0.1, 0.9, (B, 3))
    goal = np.concatenate([c - 0.05, c + 0.05], 1).astype(np.float32)
    n_obs = rng.integers(5, 61, B).astype(np.int32)
    side = rng.uniform(0.05, 0.25, (B, 64, 3))
    lo = rng.uniform(0.0, 1.0, (B, 64, 3)) * (1.0 - side)
    boxes = np.concatenate([lo, lo + side], 2).astype(np.float32)
    boxes[np.arange(64)[None, :] >= n_obs[:, None]] = 0.0
    return x0, goal, boxes, n_obs


def _conditions(B, rng):
    x0, goal, boxes, _ = _boxes_arrays(B, rng)
    return np.concatenate([x0, 0.5 * (goal[:, :3] + goal[:, 3:]), 0.5 * (goal[:, 3:] - goal[:, :3]),
                           boxes.reshape(B, -1)], 1).astype(np.float32)


def _targets(cond, rng):
    """States between start and goal, as certified plans pass through."""
    t = rng.uniform(0.0, 1.0, (len(cond), 1))
    d = cond[:, 6:9] - cond[:, :3]
    pos = cond[:, :3] + t * d + 0.08 * rng.standard_normal((len(cond), 3))
    vel = 0.3 * d + 0.15 * rng.standard_normal((len(cond), 3))
    return np.concatenate([np.clip(pos, 0, 1), np.clip(vel, -0.5, 0.5)], 1).astype(np.float32)


def _minibatches(case, seed):
    rng = _rng(seed, 20)
    out = []
    for _ in range(case["steps"]):
        c = _conditions(case["B"], rng)
        out.append((c, _targets(c, rng)))
    return out


def _prepare_net(case, seed):
    rng = _rng(seed, 20)
    if case["what"] == "train":
        mlp = _lib.MLP(case["B"])
        p = _params()
        mlp.set_state(dict(params=p, m1=np.zeros_like(p), m2=np.full_like(p, ADAM_M2), t=ADAM_T0))
        return dict(mlp=mlp, batches=[(_dev(c), _dev(z)) for c, z in _minibatches(case, seed)])
    if case["what"] == "forward":
        mlp = _lib.MLP(case["B"])
        mlp.set_params(_params())
        return dict(mlp=mlp, cond=_dev(_conditions(case["B"], rng)))
    mlp = _lib.MLP(64)
    mlp.set_params(_params())
    x0, goal, boxes, n_obs = _boxes_arrays(1, rng)
    n = case["n"]
    return dict(mlp=mlp, map=(_dev(x0), _dev(goal), _dev(boxes), torch.from_numpy(n_obs).cuda()),
                u=_dev(rng.uniform(0, 1, (1, n))), eps=_dev(rng.standard_normal((1, n, 6))))


def _run_net(st):
    mlp = st["mlp"]
    if "batches" in st:
        losses = [mlp.train_step(c, z, LEARNING_RATE) for c, z in st["batches"]]
        return dict(losses=np.asarray(losses, np.float32), params=mlp.get_params())
    if "cond" in st:
        return dict(out=mlp.forward(st["cond"]))
    cond = mlp.condition(*st["map"])
    return dict(cond=cond, states=mlp.sample(cond, st["u"], st["eps"]))


def _net64(w, x):
    at = 0
    for k, (fi, fo) in enumerate(LAYERS):
        x = x @ w[at:at + fi * fo].view(fo, fi).T + w[at + fi * fo:at + fi * fo + fo]
        at += fi * fo + fo
        if k < len(LAYERS) - 1:
            x = torch.relu(x)
    return x


def _exact_net(case, seed):
    rng = _rng(seed, 20)
    w = torch.from_numpy(_params()).double()
    if case["what"] == "forward":
        return dict(out=_net64(w, torch.from_numpy(_conditions(case["B"], rng)).double()))
    if case["what"] == "sample":
        x0, goal, boxes, _ = _boxes_arrays(1, rng)
        g = goal.astype(np.float64)
        cond = np.concatenate([x0, 0.5 * (g[:, :3] + g[:, 3:]), 0.5 * (g[:, 3:] - g[:, :3]),
                               boxes.reshape(1, -1)], 1)
        n = case["n"]
        u = rng.uniform(0, 1, (1, n)).astype(np.float32).astype(np.float64)
        eps = rng.standard_normal((1, n, 6)).astype(np.float32).astype(np.float64)
        y = _net64(w, torch.from_numpy(cond))[0].numpy()
        cdf = np.cumsum(np.exp(y[:COMPONENTS] - y[:COMPONENTS].max()))
        k = np.minimum(np.searchsorted(cdf, u[0] * cdf[-1], side="right"), COMPONENTS - 1)
        mu = y[COMPONENTS:7 * COMPONENTS].reshape(COMPONENTS, 6)[k]
        sd = np.exp(np.clip(y[7 * COMPONENTS:].reshape(COMPONENTS, 6), -4.0, 2.0))[k]
        return dict(cond=cond, states=np.clip(mu + sd * eps[0], STATE_LO, STATE_HI)[None])
    w.requires_grad_(True)
    m1, m2 = torch.zeros_like(w), torch.full_like(w, float(np.float32(ADAM_M2)))
    losses = []
    for i, (c, z) in enumerate(_minibatches(case, seed)):
        y = _net64(w, torch.from_numpy(c).double())
        B = len(c)
        mu = y[:, COMPONENTS:7 * COMPONENTS].view(B, COMPONENTS, 6)
        s = y[:, 7 * COMPONENTS:].view(B, COMPONENTS, 6).clamp(-4.0, 2.0)
        r = (torch.from_numpy(z).double()[:, None, :] - mu) * torch.exp(-s)
        a = torch.log_softmax(y[:, :COMPONENTS], 1) - (0.5 * r * r + s).sum(2) \
            - 3.0 * math.log(2.0 * math.pi)
        loss = -torch.logsumexp(a, 1).mean()
        g, = torch.autograd.grad(loss, w)
        t = ADAM_T0 + 1 + i
        with torch.no_grad():
            m1.mul_(BETA1).add_(g, alpha=1 - BETA1)
            m2.mul_(BETA2).add_(g * g, alpha=1 - BETA2)
            w -= LEARNING_RATE * (m1 / (1 - BETA1 ** t)) / ((m2 / (1 - BETA2 ** t)).sqrt() + EPS)
        losses.append(float(loss.detach()))
    return dict(losses=np.asarray(losses), params=w.detach())


# --------------------------------------------------------------------------
def prepare(case, seed):
    if case["what"] == "query":
        return _prepare_query(case, seed)
    if case["what"] == "batch":
        return _prepare_batch(case, seed)
    return _prepare_net(case, seed)


def run(state):
    if "pl" in state:
        return _run_query(state)
    if "b" in state:
        return _run_batch(state)
    return _run_net(state)


def exact(case, seed):
    if case["what"] == "query":
        return _exact_query(case, seed)
    if case["what"] == "batch":
        return None
    return _exact_net(case, seed)


def _query_work(n, N, n_obs, steps, mc):
    """Inputs read once, and the arithmetic on them: the Near bound of every
    ordered pair (27 operations), for the 5 % of pairs that connect the steering
    (150) and one range test per box (12); the deviation table; certification
    of one plan of 64 steps."""
    read = 4 * (6 * n + 6 * n_obs + 6 * steps * N + 6 * min(64, steps) * mc)
    ops = n * n * (27 + 0.05 * (150 + 12 * n_obs)) + 24 * steps * N + \
        64 * mc * (36 + 12 * n_obs)
    return read, ops


def work(case):
    if case["what"] == "query":
        b, f = _query_work(case["n"], case["N"], case["n_obs"], S_MAX, MC)
        return {"bytes": b + 24 * case["n"] * case["halton"], "flops": f}
    if case["what"] == "batch":
        steps, mc = (S_MAX, MC) if case["mixed"] else (256, 2000)
        n = (case["n_lo"] + case["n_hi"]) / 2
        # mean of n^2 over the uniform sizes
        n2 = (case["n_lo"] ** 2 + case["n_lo"] * case["n_hi"] + case["n_hi"] ** 2) / 3
        b, f = _query_work(n, 128, 33, steps, mc)
        f += (n2 - n * n) * (27 + 0.05 * (150 + 12 * 33))
        return {"bytes": case["q"] * b, "flops": case["q"] * f}
    weights = sum(i * o + o for i, o in LAYERS)
    rows = 1 if case["what"] == "sample" else case["B"]
    if case["what"] == "train":
        # parameters and both moments read and written, inputs read
        return {"bytes": case["steps"] * (24 * weights + 4 * rows * (NET_IN + 6)),
                "flops": case["steps"] * 6.0 * rows * weights}
    if case["what"] == "forward":
        return {"bytes": 2 * weights + 4 * rows * (NET_IN + NET_OUT), "flops": 2.0 * rows * weights}
    return {"bytes": 2 * weights + 4 * (2 * NET_IN + case["n"] * 13),
            "flops": 2.0 * weights + 40.0 * case["n"]}
