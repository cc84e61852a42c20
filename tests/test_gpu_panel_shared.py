"""Block panels whose neighbouring lanes share a block's values: the widths at which the number of sharing
lanes changes (4 columns: none, 8: two, 16 and more: four), padded and full, and the widest, against
single solves: two PCG iterations, both V-cycle precisions, whole sweeps and groups.  Other orders of
the same sums: 1e-11 relative in FP64, 1e-5 with the FP32 V-cycle."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("tail", [0, 4096])
@pytest.mark.parametrize("cols", [3, 4, 5, 8, 15, 16, 33, 64])
def test_panel_columns_equal_single_solves(cols, tail):
    p = make_problem(13, ny=11, nz=12, nu=0.3)
    h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                    E.eamg_default_setup_params(vcycle_fp32=1, dense_tail_dofs=tail, coarsest_max_dofs=60))
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
    B = torch.tensor(np.random.default_rng(cols).standard_normal((cols, p.n_dofs)), device="cuda") * free
    for prec, tol in ((E.EAMG_PRECOND_VCYCLE, 1e-11), (E.EAMG_PRECOND_VCYCLE_FP32, 1e-5)):
        kw = dict(rtol=0.0, max_it=2, precond=prec)
        X = h.solve_batch(B, **kw)[0]
        for c in (0, cols // 2, cols - 1):
            x = h.solve(B[c], **kw)[0]
            err = float((X[c] - x).norm() / x.norm())
            print(f"\n[{cols} columns, tail {tail}, precond {prec}, column {c}] {err:.1e}", flush=True)
            assert err <= tol
    h.close()
