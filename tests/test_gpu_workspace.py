"""Device memory of a context and of a batch's slots: only the half-space model's
hold the queue of 32 bytes a candidate pair, only the box model's the rank
tables."""

import pytest

from paper_1607_06886_amd import _lib
from tests._gpu import print_case

pytestmark = pytest.mark.gpu

N, S, Q = 32, 64, 1 << 22
TABLES = 3 * (S + 1) * (6 * N + (N + 1) * N // 8)   # rank rows and prefix sets (rank_tables.hpp)
GRAIN = 4 << 20                                     # an allocation's rounding


def _taken(make):
    import torch
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    obj = make()
    taken = free - torch.cuda.mem_get_info()[0]
    obj.close()
    return taken


@pytest.mark.parametrize("slots", [0, 3])
def test_the_pair_queue_is_the_half_space_models(slots):
    print_case("workspace", slots=slots)
    import torch
    torch.zeros(1, device="cuda")
    cfg = dict(n_particles=N, max_nodes=200, max_obstacles=8, max_steps=S, mc_particles=256, cap_plans=1 << 16,
               cap_pairs=Q, cap_edges=1 << 18)
    make = (lambda m: _lib.Batch(slots, cp_model=m, **cfg)) if slots else (lambda m: _lib.Planner(cp_model=m, **cfg))
    make(0).close()                                 # (what the first one alone takes)
    box, half = _taken(lambda: make(0)), _taken(lambda: make(1))
    print("  MB", box >> 20, half >> 20, flush=True)
    n = max(slots, 1)
    assert half - box >= n * (32 * Q - TABLES) - GRAIN
