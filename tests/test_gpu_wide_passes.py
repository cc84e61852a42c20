"""The dense V-cycle tail built in passes narrower than the device's memory allows, as where the panels of a
full pass do not fit: passes of one slice of 128 columns, of a slice and two columns, of fewer, and with a
last pass of two columns.  A column of the tail takes the same operations in any pass, so V-cycles agree
with those of the full pass to rounding (1e-14), and with the same hierarchy's sparse V-cycle to 1e-11
(sums of a few hundred terms)."""
import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "poisson": dict(n=21, ny=17, nz=19, kind="poisson", clamp="all"),
    "elasticity": dict(n=9, ny=7, nz=8, nu=0.35),
}


@pytest.mark.parametrize("name", list(CASES))
def test_narrow_passes_build_the_same_tail(name, monkeypatch):
    p = make_problem(**CASES[name])
    r = np.random.default_rng(8).standard_normal(p.n_dofs)
    r[np.repeat(p.dirichlet.astype(bool), p.dim)] = 0.0

    def vcycle(dofs, cols=None):
        if cols:
            monkeypatch.setenv("EAMG_WIDE_COLS", str(cols))
        h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                        E.eamg_default_setup_params(dense_tail_dofs=dofs, coarsest_max_dofs=60))
        monkeypatch.delenv("EAMG_WIDE_COLS", raising=False)
        n = E.eamg_dense_tail(h.h)[1]
        z = torch.empty(p.n_dofs, dtype=torch.float64, device="cuda")
        E.eamg_vcycle(h.h, torch.tensor(r, device="cuda"), z)
        torch.cuda.synchronize()
        h.close()
        return z.cpu().numpy(), n

    sparse, _ = vcycle(0)
    full, n = vcycle(16384)
    print(f"\n[{name}] tail of {n} dofs", flush=True)
    assert n > 260
    for cols in (128, 130, 64, 34, (n - 1) // 2 * 2):
        z, m = vcycle(16384, cols)
        err, same = (np.linalg.norm(z - y) / np.linalg.norm(y) for y in (sparse, full))
        print(f"    {cols} columns a pass, {(n - 1) % cols + 1} in the last: {err:.1e}, {same:.1e}", flush=True)
        assert m == n and err <= 1e-11 and same <= 1e-14
