"""Grouped sweep stages (plan_sweeps, k_group_rhs, k_gs_group, k_group_fill, and their panel forms)
against the general path, the colour-by-colour sweeps with which a dense tail is built: two PCG
iterations by eamg_solve and by eamg_solve_batch on a hierarchy without a tail (every level's sweeps
grouped where the plan says so) and on the same hierarchy with the tail on its first coarse level.
The cases give levels that are one group, several groups, groups beside single colours, and
pseudo-inverted (singular) diagonal blocks; blocks of 1, 3 and 6; every row-team shape; panels of 1 and
9 columns.  Both orders sum the same products: FP64 1e-11 relative (a few hundred terms a row, recursion
depth a few tens), FP32 V-cycle 1e-5 as elsewhere."""
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


def _hierarchy(p, tail, **kw):
    return E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                       E.eamg_default_setup_params(vcycle_fp32=1, dense_tail_dofs=tail, **kw))


def _compare(p, h, ref, seed):
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
    B = torch.tensor(np.random.default_rng(seed).standard_normal((9, p.n_dofs)), device="cuda") * free
    errs = {}
    for prec, tol in ((E.EAMG_PRECOND_VCYCLE, 1e-11), (E.EAMG_PRECOND_VCYCLE_FP32, 1e-5)):
        kw = dict(rtol=0.0, max_it=2, precond=prec)
        x0 = ref.solve(B[0], **kw)[0]
        xs = [h.solve(B[0], **kw)[0], h.solve_batch(B[:1], **kw)[0][0], h.solve_batch(B, **kw)[0][0]]
        errs[prec] = [float((x - x0).norm() / x0.norm()) for x in xs]
        assert max(errs[prec]) <= tol, (prec, errs)
    return errs


@pytest.mark.parametrize("name", list(CASES))
def test_grouped_sweeps_equal_colour_sweeps(name):
    p = make_problem(**CASES[name])
    h, ref = _hierarchy(p, 0, coarsest_max_dofs=60), _hierarchy(p, 16384, coarsest_max_dofs=60)
    colours = [E.eamg_level_info_get(h.h, l)["n_colors"] for l in range(h.stats()["n_levels"])]
    print(f"\n[{name}] colours {colours} {_compare(p, h, ref, 5)}", flush=True)
    h.close()
    ref.close()


@pytest.mark.parametrize("group", [8, 64, 128, 256])
@pytest.mark.parametrize("name", ["poisson", "elasticity"])
def test_grouped_sweeps_with_every_row_team(name, group, monkeypatch):
    p = make_problem(**CASES[name])
    h, ref = _hierarchy(p, 0), _hierarchy(p, 16384)
    monkeypatch.setitem(os.environ, "EAMG_FORCE_GROUP", str(group))
    E.eamg_autotune(h.h, 0)
    print(f"\n[{name}, {group} lanes] {_compare(p, h, ref, 6)}", flush=True)
    h.close()
    ref.close()
