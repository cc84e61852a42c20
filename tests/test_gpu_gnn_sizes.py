"""Edge-network kernels at the edges of their tiles and chunks (32-edge tiles, four edges per
wavefront, 2048-edge chunks): logits, loss and gradients against the
float64 oracle network, with the bars of test_gpu_gnn.py."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from oracle import gnn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 3, 5, 31, 32, 33, 2047, 2049, 4097])
def test_sizes(m):
    rng = np.random.default_rng(m)
    n = max(2, m // 3)
    u = rng.integers(0, n, size=m)
    v = (u + rng.integers(1, n, size=m)) % n if n > 2 else 1 - u
    edges = np.sort(np.stack([u, v], axis=1), axis=1).astype(np.int32)
    X = rng.standard_normal((m, gnn.F)).astype(np.float32)
    y = (rng.random(m) < 0.5).astype(np.float32)
    w = rng.uniform(0.2, 1.0, m).astype(np.float32)
    p = gnn.init_params(3)
    for k in p:
        if k.startswith("b"):
            p[k] = 0.05 * rng.standard_normal(p[k].shape)
    flat = np.concatenate([np.asarray(p[k], dtype=np.float64).ravel() for k in gnn.PARAM_SHAPES]).astype(np.float32)
    q, o = {}, 0
    for k, shp in gnn.PARAM_SHAPES.items():
        sz = int(np.prod(shp))
        q[k] = flat[o:o + sz].astype(np.float64).reshape(shp)
        o += sz
    net = E.EdgeNet(flat)
    z = net.forward(X, edges, n)
    loss, g = net.loss_grad(X, edges, n, y, w)
    loss2, g2 = net.loss_grad(X, edges, n, y, w)
    net.close()
    assert loss == loss2 and np.array_equal(g, g2)
    zo, _ = gnn.forward(q, X.astype(np.float64), edges, n)
    lo, go, _ = gnn.loss_and_grads(q, X.astype(np.float64), edges, n, y, weight=w)
    assert np.abs(z - zo).max() <= 2e-5 * np.abs(zo).max()
    assert abs(loss - lo) <= 1e-5 * abs(lo)
    o = 0
    for k, shp in gnn.PARAM_SHAPES.items():
        sz = int(np.prod(shp))
        ref = np.asarray(go[k]).ravel()
        assert np.abs(g[o:o + sz] - ref).max() <= 1e-4 * np.abs(ref).max() + 1e-9, k
        o += sz
