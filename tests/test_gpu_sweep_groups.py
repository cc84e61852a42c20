"""Grouped sweep stages (plan_sweeps, k_group_rhs, k_gs_group, k_group_fill) against the general
path, the colour-by-colour sweeps that the block panels run: two PCG iterations of one right-hand
side by eamg_solve and by eamg_solve_batch on the same hierarchy.  The cases give levels that are one
group, several groups, groups beside single colours, and pseudo-inverted (singular) diagonal blocks;
blocks of 1, 3 and 6; every row-team shape.  Both orders sum the same products: FP64 1e-11 relative
(a few hundred terms a row, recursion depth a few tens), FP32 V-cycle 1e-5 as elsewhere."""
import os

import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "poisson": dict(n=33, ny=29, nz=31, kind="poisson", clamp="all"),
    "poisson_flat": dict(n=64, ny=5, nz=3, kind="poisson"),
    "elasticity": dict(n=24, ny=19, nz=21, nu=0.3),
    "inclusions": dict(n=16, inclusions=5, geometry_seed=3),
    "tiny": dict(n=4, ny=3, nz=3),
}


def _compare(p, h, seed):
    b = np.random.default_rng(seed).standard_normal(p.n_dofs)
    b[np.repeat(p.dirichlet.astype(bool), p.dim)] = 0.0
    bd = torch.tensor(b, device="cuda")
    errs = {}
    for prec, tol in ((E.EAMG_PRECOND_VCYCLE, 1e-11), (E.EAMG_PRECOND_VCYCLE_FP32, 1e-5)):
        x, _ = h.solve(bd, rtol=0.0, max_it=2, precond=prec)
        X, _, _ = h.solve_batch(bd[None], rtol=0.0, max_it=2, precond=prec)
        err = float((x - X[0]).norm() / X[0].norm())
        errs[prec] = err
        assert err <= tol, (prec, err)
    return errs


@pytest.mark.parametrize("name", list(CASES))
def test_grouped_sweeps_equal_colour_sweeps(name):
    p = make_problem(**CASES[name])
    h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                    E.eamg_default_setup_params(vcycle_fp32=1, coarsest_max_dofs=60))
    colours = [E.eamg_level_info_get(h.h, l)["n_colors"] for l in range(h.stats()["n_levels"])]
    print(f"\n[{name}] colours {colours} {_compare(p, h, 5)}", flush=True)
    h.close()


@pytest.mark.parametrize("group", [8, 64, 128, 256])
@pytest.mark.parametrize("name", ["poisson", "elasticity"])
def test_grouped_sweeps_with_every_row_team(name, group, monkeypatch):
    p = make_problem(**CASES[name])
    h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                    E.eamg_default_setup_params(vcycle_fp32=1))
    monkeypatch.setitem(os.environ, "EAMG_FORCE_GROUP", str(group))
    E.eamg_autotune(h.h, 0)
    print(f"\n[{name}, {group} lanes] {_compare(p, h, 6)}", flush=True)
    h.close()
