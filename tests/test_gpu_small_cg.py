"""The CG kernels of small systems (one workgroup for the x and r update and the stopping test; the
direction formed inside the SpMV; r.z summed by the last sweep launch of a level that is one group)
against the block CG, which has kernels of its own: sizes at the edges of the two rules, blocks of 1 and
3, both V-cycle precisions and no preconditioner, with and without an x0.  The same recurrences with the
sums in another order: 1e-11 relative after three iterations, 1e-5 with the FP32 V-cycle, as for the
other orders of the V-cycle's sums."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "one_workgroup": dict(n=16, ny=16, nz=6, kind="poisson"),       # 1,536 dofs, the last of that rule
    "two_launches": dict(n=17, ny=13, nz=7, kind="poisson"),        # 1,547
    "elasticity_512": dict(n=8, ny=8, nz=8, nu=0.3),                # 1,536 in blocks of 3
    "elasticity_576": dict(n=9, ny=8, nz=8, nu=0.3),
    "direction_in_spmv": dict(n=64, ny=32, nz=32, kind="poisson"),  # 65,536, the last of that rule
    "direction_apart": dict(n=65, ny=32, nz=32, kind="poisson"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_cg_equals_block_cg(name):
    p = make_problem(**CASES[name])
    h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                    E.eamg_default_setup_params(vcycle_fp32=1, coarsest_max_dofs=60))
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.n_dofs // len(p.dirichlet)), device="cuda")
    b, x0 = torch.tensor(np.random.default_rng(3).standard_normal((2, p.n_dofs)), device="cuda") * free
    for prec, tol in ((E.EAMG_PRECOND_VCYCLE, 1e-11), (E.EAMG_PRECOND_VCYCLE_FP32, 1e-5),
                      (E.EAMG_PRECOND_NONE, 1e-11)):
        kw = dict(rtol=0.0, max_it=3, precond=prec)
        for guess in (0, 1):
            x, info = h.solve(b, x=x0.clone(), use_x0=guess, **kw)
            ref = h.solve_batch(b[None], X=x0[None].clone(), use_x0=guess, **kw)[0][0]
            err = float((x - ref).norm() / ref.norm())
            print(f"\n[{name}] {p.n_dofs} dofs, precond {prec}, x0 {guess}: {err:.1e}, "
                  f"|r|/|b| {info['rel_res_true']:.1e}", flush=True)
            assert err <= tol
    h.close()
