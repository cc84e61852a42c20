"""mu_g on the device at the edges of its batches of pseudo-inverses, 32 outside neighbours at a time: on a
complete graph of n vertices every outside neighbour of a union meets all its members, so a pair has
n - 2 of them.  Against the host's code bit for bit (the same operations without contraction)."""
import numpy as np
import pytest

import paper_2011_13325_amd as E

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 6])
@pytest.mark.parametrize("n", [3, 33, 34, 35, 66, 67])
def test_mu_g_at_batch_edges(n, k):
    rng = np.random.default_rng(n)
    i, j = np.triu_indices(n, 1)
    edges = np.stack([i, j], 1).astype(np.int32)
    # positive semidefinite, of every rank up to k, so that the pseudo-inverses drop directions too
    W = []
    for e in range(len(edges)):
        b = rng.standard_normal((k, 1 + e % k))
        W.append(b @ b.T)
    M = np.einsum("nab,ncb->nac", *(2 * [rng.standard_normal((n, k, 1))])) * (rng.random((n, 1, 1)) < 0.5)
    unions = [[a, b, -1, -1] for a, b in edges[:: max(1, len(edges) // 12)]]
    if n <= 50:   # the device holds 192 entries of outside neighbours
        unions += [sorted(rng.choice(n, size=m, replace=False).tolist()) + [-1] * (4 - m)
                   for m in (1, 3, 4) for _ in range(4) if m <= n]
    u = np.array(unions, dtype=np.int32)
    dev, host = (E.eamg_criteria_eval(k, _coords(n), edges, np.array(W), M, edges[:1], u, use_device=d)[1]
                 for d in (True, False))
    print(f"\n[{n} vertices, k {k}] {len(u)} unions, {np.isfinite(host).sum()} finite", flush=True)
    np.testing.assert_array_equal(dev, host)
    assert not np.isnan(host).any()


def _coords(n):
    return np.random.default_rng(1).random((n, 3))
