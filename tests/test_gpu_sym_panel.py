"""The panel product with the packed symmetric tail (k_dense_panel_sym) over its column and tile
edges: panels of 1 to 64 columns (one and two 16-column tiles, two passes), tails of less than one
128 tile, of a ragged last tile, and of more tiles than one run.  Two PCG iterations of a batch against
the same hierarchy without a tail: the same operator, FP64 sums of up to 10^4 terms a row (1e-11
relative), FP32 V-cycle 1e-5 as elsewhere."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "one_tile": dict(n=9, ny=8, nz=8, kind="poisson", clamp="all"),
    "poisson_odd": dict(n=23, ny=19, nz=21, kind="poisson", clamp="all"),
    "elasticity": dict(n=17, ny=15, nz=13, nu=0.3),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tail_panel_equals_sparse(name):
    p = make_problem(**CASES[name])
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
    hs = [E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                      E.eamg_default_setup_params(dense_tail_dofs=d, coarsest_max_dofs=20, vcycle_fp32=1))
          for d in (0, 16384)]
    lvl, n = E.eamg_dense_tail(hs[1].h)
    print(f"\n[{name}] tail on level {lvl}, {n} dofs", flush=True)
    assert lvl >= 1 and (n < 128) == (name == "one_tile")
    for m in (1, 2, 4, 7, 16, 17, 32, 40):
        B = torch.tensor(np.random.default_rng([3, m]).standard_normal((m, p.n_dofs)), device="cuda") * free
        for prec, tol in ((E.EAMG_PRECOND_VCYCLE, 1e-11), (E.EAMG_PRECOND_VCYCLE_FP32, 1e-5)):
            X = [h.solve_batch(B, rtol=0.0, max_it=2, precond=prec)[0] for h in hs]
            err = float(((X[1] - X[0]).norm(dim=1) / X[0].norm(dim=1)).max())
            assert err <= tol, (m, prec, err)
    for h in hs:
        h.close()
