"""Outputs of the proposal network written over its own condition rows: the
same values as into memory of their own, wherever the outputs begin."""

import ctypes

import numpy as np
import pytest

from paper_1607_06886_amd import _lib
from tests._gpu import print_case

pytestmark = pytest.mark.gpu


# rows: one workgroup, more rows than one pass over the compute units takes
# (16 x 256), and its double; outputs from the first condition row on, from the
# middle and so that only the last condition row is met
@pytest.mark.parametrize("B", [5, 5000, 9000])
@pytest.mark.parametrize("at", ["first", "middle", "last"])
def test_outputs_over_conditions(B, at):
    print_case("proposal overlap", B=B, at=at)
    import torch
    rng = np.random.default_rng(B)
    cond = torch.from_numpy(rng.uniform(-1, 1, (B, 396)).astype(np.float32)).cuda()
    mlp = _lib.MLP(B)
    mlp.set_params(rng.standard_normal(mlp.n_params).astype(np.float32) * 0.05)
    want = mlp.forward(cond).cpu()
    start = {"first": 0, "middle": (B // 2) * 396, "last": B * 396 - 7}[at]
    buf = torch.zeros(B * 396 + B * 208, dtype=torch.float32, device="cuda")
    buf[:B * 396] = cond.flatten()
    torch.cuda.synchronize()
    mlp._check(mlp.lib.pump_mlp_forward(mlp.m, buf.data_ptr(), B, ctypes.c_void_p(buf.data_ptr() + 4 * start), 1))
    got = buf[start:start + B * 208].view(B, 208).cpu()
    assert torch.equal(got, want)
    # what the outputs do not cover is as it was
    flat = cond.flatten().cpu()
    assert torch.equal(buf[:min(start, B * 396)].cpu(), flat[:min(start, B * 396)])
    if start + B * 208 < B * 396:
        assert torch.equal(buf[start + B * 208:B * 396].cpu(), flat[start + B * 208:])
    mlp.close()
