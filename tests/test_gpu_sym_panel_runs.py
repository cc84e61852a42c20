"""The panel product with the packed symmetric tail where a workgroup takes a run of several tiles: two from
11,521 dofs on, four from 16,257, up to the largest tail (16,384), with ragged last runs and a ragged last
tile.  Two PCG iterations of a batch against the same hierarchy without a tail: the same operator, FP64
sums of up to 2 x 10^4 terms a row (1e-11 relative), FP32 V-cycle 1e-5 as elsewhere."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "two_tiles_a_run": (dict(n=37, ny=29, nz=33, nu=0.35),
                        dict(cap_std_l0=6, cap_std=4, cap_aux=4, sigma=18.0), 11520, 16256),
    "four_tiles_a_run": (dict(n=43, ny=44, nz=40, kind="poisson", clamp="all"), {}, 16256, 16384),
}


@pytest.mark.parametrize("name", list(CASES))
def test_runs_of_tiles_equal_the_sparse_vcycle(name):
    mesh, prm, above, upto = CASES[name]
    p = make_problem(**mesh)
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
    hs = [E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                      E.eamg_default_setup_params(dense_tail_dofs=d, vcycle_fp32=1, **prm)) for d in (0, 16384)]
    n = E.eamg_dense_tail(hs[1].h)[1]
    print(f"\n[{name}] tail of {n} dofs", flush=True)
    assert above < n <= upto and n % 128
    for m in (1, 7, 16, 40):
        B = torch.tensor(np.random.default_rng([4, m]).standard_normal((m, p.n_dofs)), device="cuda") * free
        for prec, tol in ((E.EAMG_PRECOND_VCYCLE, 1e-11), (E.EAMG_PRECOND_VCYCLE_FP32, 1e-5)):
            X = [h.solve_batch(B, rtol=0.0, max_it=2, precond=prec)[0] for h in hs]
            err = float(((X[1] - X[0]).norm(dim=1) / X[0].norm(dim=1)).max())
            print(f"    {m} columns, precond {prec}: {err:.1e}", flush=True)
            assert err <= tol, (m, prec, err)
    for h in hs:
        h.close()
