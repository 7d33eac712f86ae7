"""The proposal network's kernels at the edges of their tiles: 16 and 32 batch
rows a workgroup (the latter beyond 4096 rows), the last k-step of a weight
gradient, workgroups of 256 draws.

Rows do not depend on one another and every product is one chain in k order,
so a batch equals its parts bit by bit.  A gradient element may differ from
the FP64 oracle's by one BF16 rounding (2^-8) of a back-propagated value and
one of a layer input taken the other way: 2^-7 of the layer's largest
gradient, on average 2^-9 of its mean magnitude."""

import numpy as np
import pytest

from oracle import proposal as pp
from paper_1607_06886_amd import _lib
from tests._gpu import print_case
from tests.test_gpu_proposal import _inputs, flat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 33, 4095, 4096, 4129])
def test_forward_rows_do_not_depend_on_the_batch(B):
    print_case("mlp_forward_tiles", B=B)
    m = _lib.MLP(B)
    m.set_params(flat(pp.init_params(3)))
    X, _ = _inputs(B, B)
    y = m.forward(X)
    parts = np.concatenate([m.forward(X[i:i + 1001]) for i in range(0, B, 1001)])
    assert np.isfinite(y).all() and np.array_equal(y, parts)
    tail = m.forward(X[-1:])
    assert np.array_equal(y[-1:], tail)
    m.close()


@pytest.mark.parametrize("B", [1, 16, 17, 31, 33, 257, 545])
def test_gradients_at_tile_edges(B):
    print_case("mlp_grad_tiles", B=B)
    params = pp.init_params(21)
    X, Z = _inputs(100 + B, B)
    m = _lib.MLP(600)
    m.set_params(flat(params))
    m.loss_grad(*_inputs(7, 600))        # the rows past the batch held something
    loss, g = m.loss_grad(X, Z)
    y, cache = pp.forward(params, X, bf16_ops=True)
    want = flat(pp.backward(params, cache, pp.nll_grad(y, Z), bf16_ops=True)).astype(np.float64)
    lref = pp.nll(y, Z)
    assert abs(loss - lref) <= 1e-2 * abs(lref) + 1e-3
    o = 0
    for li, (fi, fo) in enumerate(pp.LAYERS):
        for n in (fi * fo, fo):
            a, b = g[o:o + n].astype(np.float64), want[o:o + n]
            assert np.abs(a - b).max() <= 2.0 ** -7 * np.abs(b).max(), li
            assert np.abs(a - b).mean() <= 2.0 ** -9 * np.abs(b).mean(), li
            o += n
    m.close()


@pytest.mark.parametrize("q, n", [(1, 1), (2, 255), (3, 256), (1, 257), (5, 1025)])
def test_samples_at_workgroup_edges(q, n):
    print_case("mlp_sample_tiles", q=q, n=n)
    rng = np.random.default_rng(q * n)
    params = [(np.zeros((fo, fi), np.float32), np.zeros(fo, np.float32)) for fi, fo in pp.LAYERS]
    yb = rng.normal(0, 1.0, pp.D_OUT).astype(np.float32)
    yb[112:] = rng.uniform(-4, -1, 96)
    params[-1] = (params[-1][0], yb)
    m = _lib.MLP(8)
    m.set_params(flat(params))
    cond = rng.uniform(0, 1, (q, pp.D_IN)).astype(np.float32)
    u = rng.uniform(0, 1, (q, n)).astype(np.float32)
    u[0, 0], u[-1, -1] = 0.0, np.float32(1.0) - np.float32(2.0 ** -24)
    eps = rng.standard_normal((q, n, 6)).astype(np.float32)
    out = m.sample(cond, u, eps)
    for i in range(q):
        z, _ = pp.sample(yb.astype(np.float64), u[i].astype(np.float64), eps[i].astype(np.float64))
        np.testing.assert_allclose(out[i], z, rtol=0, atol=4e-6)
    m.close()
