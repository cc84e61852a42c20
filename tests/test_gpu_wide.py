"""The dense V-cycle tail's construction by wide panels (wide.hip) at the edges of its launches:
an odd number of columns, one dof per vertex, the last columns of a slice, and more columns than
one pass takes (8192).  The V-cycle with the tail against the same hierarchy's sparse V-cycle: the
same linear map, both in FP64 with sums of a few hundred terms, so 1e-11 relative leaves four
digits over rounding."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "poisson_small_odd": dict(n=13, ny=11, nz=9, kind="poisson", clamp="all"),
    "poisson_two_passes": dict(n=40, ny=37, nz=35, kind="poisson", clamp="all"),
    "elasticity_ragged": dict(n=9, ny=7, nz=8, nu=0.35),
    "elasticity_two_passes": dict(n=21, ny=20, nz=19, nu=0.3),
}
PASS = 8192


@pytest.mark.parametrize("name", list(CASES))
def test_wide_tail_equals_sparse_vcycle(name):
    p = make_problem(**CASES[name])
    z = {}
    for dofs in (0, 16384):
        h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                        E.eamg_default_setup_params(dense_tail_dofs=dofs, coarsest_max_dofs=60))
        lvl, n = E.eamg_dense_tail(h.h)
        assert (lvl >= 1) == (dofs > 0)
        if dofs:
            print(f"\n[{name}] tail on level {lvl}, {n} dofs", flush=True)
            assert (n > PASS) == name.endswith("two_passes")
        r = np.random.default_rng(7).standard_normal(p.n_dofs)
        r[np.repeat(p.dirichlet.astype(bool), p.dim)] = 0.0
        out = torch.empty(p.n_dofs, dtype=torch.float64, device="cuda")
        E.eamg_vcycle(h.h, torch.tensor(r, device="cuda"), out)
        torch.cuda.synchronize()
        z[dofs] = out.cpu().numpy()
        h.close()
    err = np.linalg.norm(z[16384] - z[0]) / np.linalg.norm(z[0])
    print(f"[{name}] relative difference {err:.2e}", flush=True)
    assert err <= 1e-11
