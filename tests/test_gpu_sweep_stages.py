"""Sweeps whose colours run as groups against the same sweeps with every colour launched on its own (the
same hierarchy set up without memory for groups, EAMG_GROUP_MB = 0), and setups whose memory holds the
groups of some levels only.  Both orders sum the same products: FP64 1e-11 relative (a few hundred terms a
row, recursion depth a few tens), FP32 V-cycle 1e-5 as elsewhere."""
import re

import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "poisson": dict(n=33, ny=29, nz=31, kind="poisson", clamp="all"),
    "elasticity": dict(n=13, ny=12, nz=14, nu=0.3),
}
# layouts of the levels, by block size: one group, several groups, groups beside single colours
LAYOUTS = {
    "poisson": (CASES["poisson"], {(1, "one"), (1, "several")}),
    "poisson_flat": (dict(n=64, ny=5, nz=3, kind="poisson"), {(1, "one")}),
    "elasticity": (dict(n=24, ny=19, nz=21, nu=0.3), {(3, "one"), (6, "one"), (6, "several")}),
    "elasticity_beside": (dict(n=30, ny=29, nz=31, nu=0.3), {(3, "beside"), (6, "one"), (6, "several")}),
    # singular (pseudo-inverted) diagonal blocks
    "inclusions": (dict(n=16, inclusions=5, geometry_seed=3), {(3, "one"), (6, "one"), (6, "several")}),
}
STAGE = re.compile(r"L(\d+) c(\d+)(?:-(\d+))? k_gs_color<double, (\d), true>( grouped)?$")
F64, F32 = E.EAMG_PRECOND_VCYCLE, E.EAMG_PRECOND_VCYCLE_FP32


def _hierarchy(p, monkeypatch, megabytes=None, **kw):
    if megabytes is not None:
        monkeypatch.setenv("EAMG_GROUP_MB", str(megabytes))
    h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                    E.eamg_default_setup_params(vcycle_fp32=1, **kw))
    monkeypatch.delenv("EAMG_GROUP_MB", raising=False)
    return h


def _rhs(p, m, seed):
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
    return torch.tensor(np.random.default_rng(seed).standard_normal((m, p.n_dofs)), device="cuda") * free


def _stages(p, h):
    """{level: [(first colour, last colour) of every forward stage]} and the levels' block sizes."""
    E.eamg_profile_enable(h.h, 3)
    E.eamg_vcycle(h.h, _rhs(p, 1, 0)[0], torch.empty(p.n_dofs, dtype=torch.float64, device="cuda"))
    out, bs = {}, {}
    for k in E.eamg_profile_read(h.h, 4096):
        if m := STAGE.match(k["name"]):
            out.setdefault(int(m[1]), []).append((int(m[2]), int(m[3] or m[2])))
            bs[int(m[1])] = int(m[4])
    E.eamg_profile_enable(h.h, False)
    return {l: sorted(v) for l, v in out.items()}, bs


def _groups(stages):
    return sum(c1 > c0 for v in stages.values() for c0, c1 in v)


def _compare(p, h, ref, seed=5, rhs=9):
    B = _rhs(p, rhs, seed)
    for prec, tol in ((F64, 1e-11), (F32, 1e-5)):
        kw = dict(rtol=0.0, max_it=2, precond=prec)
        x0, X0 = ref.solve(B[0], **kw)[0], ref.solve_batch(B, **kw)[0]
        X = h.solve_batch(B, **kw)[0]
        errs = [float((h.solve(B[0], **kw)[0] - x0).norm() / x0.norm()),
                float((h.solve_batch(B[:1], **kw)[0][0] - x0).norm() / x0.norm()),
                float(((X - X0).norm(dim=1) / X0.norm(dim=1)).max())]
        z, z0 = torch.empty_like(x0), torch.empty_like(x0)
        E.eamg_vcycle(h.h, B[1], z, precision=prec)
        E.eamg_vcycle(ref.h, B[1], z0, precision=prec)
        errs.append(float((z - z0).norm() / z0.norm()))
        print(f"    {errs}", flush=True)
        assert max(errs) <= tol, (prec, errs)


def _layouts(stages, bs):
    out = set()
    for l, v in stages.items():
        groups = sum(c1 > c0 for c0, c1 in v)
        if groups:
            out.add((bs[l], "one" if len(v) == 1 else "several" if groups == len(v) else "beside"))
    return out


@pytest.mark.parametrize("name", list(LAYOUTS))
def test_groups_equal_single_colours(name, monkeypatch):
    mesh, want = LAYOUTS[name]
    p = make_problem(**mesh)
    h, ref = (_hierarchy(p, monkeypatch, mb, coarsest_max_dofs=60) for mb in (None, 0))
    stages, bs = _stages(p, h)
    print(f"\n[{name}] {stages}", flush=True)
    assert want <= _layouts(stages, bs) and not _groups(_stages(p, ref)[0])
    _compare(p, h, ref)
    h.close()
    ref.close()


@pytest.mark.parametrize("group", [8, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("name", ["poisson", "elasticity"])
def test_groups_with_every_row_team_equal_single_colours(name, group, monkeypatch):
    p = make_problem(**LAYOUTS[name][0])
    h, ref = (_hierarchy(p, monkeypatch, mb) for mb in (None, 0))
    monkeypatch.setenv("EAMG_FORCE_GROUP", str(group))
    E.eamg_autotune(h.h, 0)
    monkeypatch.delenv("EAMG_FORCE_GROUP")
    assert _groups(_stages(p, h)[0])
    _compare(p, h, ref)
    h.close()
    ref.close()


@pytest.mark.parametrize("name", list(CASES))
def test_setup_without_memory_for_groups_runs_colour_by_colour(name, monkeypatch):
    p = make_problem(**CASES[name])
    full = _hierarchy(p, monkeypatch)
    want, _ = _stages(p, full)
    none = _hierarchy(p, monkeypatch, 0)
    for mb in (1, 2, 4, 8, 16, 32, 64):   # the first that holds the groups of some level
        part = _hierarchy(p, monkeypatch, mb)
        if _groups(_stages(p, part)[0]):
            break
        part.close()
    got0, gotp = _stages(p, none)[0], _stages(p, part)[0]
    print(f"\n[{name}] groups {_groups(want)}, {_groups(gotp)} in little memory, {_groups(got0)} in none", flush=True)
    colours = {l: v[-1][1] + 1 for l, v in want.items()}
    assert _groups(want) and got0 == {l: [(c, c) for c in range(n)] for l, n in colours.items()}
    for l, n in colours.items():   # a level has all its groups or none
        assert gotp[l] in (want[l], got0[l]), l
    assert 0 < _groups(gotp) < _groups(want)
    _compare(p, part, none)
    b = _rhs(p, 1, 3)[0]
    its = [h.solve(b, precond=prec)[1]["iterations"] for h in (full, part, none) for prec in (F64, F32)]
    assert max(its) - min(its) <= 1, its
    monkeypatch.setenv("EAMG_GROUP_MB", "0")
    f0 = E.Fused([full, part], dense_tail_dofs=0)
    monkeypatch.delenv("EAMG_GROUP_MB")
    f = E.Fused([full, part], dense_tail_dofs=0)
    for prec, tol in ((F64, 1e-11), (F32, 1e-5)):
        kw = dict(rtol=0.0, max_it=2, precond=prec)
        for x, x0 in zip(f.solve([b, b], **kw)[0], f0.solve([b, b], **kw)[0]):
            assert float((x - x0).norm() / x0.norm()) <= tol
    for h in (f, f0, full, none, part):
        h.close()


@pytest.mark.parametrize("name", list(CASES))
def test_coarsest_level_the_coarsening_stalled_on_has_no_sweeps(name, monkeypatch):
    # a bound no level reaches: the last level was planned for sweeps before its matching found nothing
    p = make_problem(**CASES[name])
    h = _hierarchy(p, monkeypatch, coarsest_max_dofs=1)
    ref = _hierarchy(p, monkeypatch, 0, coarsest_max_dofs=1)
    levels = h.stats()["n_levels"]
    assert sorted(_stages(p, h)[0]) == list(range(levels - 1))
    _compare(p, h, ref)
    h.close()
    ref.close()


@pytest.mark.parametrize("name", list(CASES))
def test_panels_without_memory_for_groups_run_colour_by_colour(name, monkeypatch):
    p = make_problem(**CASES[name])
    h, ref = _hierarchy(p, monkeypatch), _hierarchy(p, monkeypatch)
    B = _rhs(p, 5, 7)
    for prec, tol in ((F64, 1e-11), (F32, 1e-5)):
        kw = dict(rtol=0.0, max_it=2, precond=prec)
        names = {}
        for key, hier in (("groups", ref), ("none", h)):
            if key == "none":
                monkeypatch.setenv("EAMG_GROUP_MB", "0")
            X = hier.solve_batch(B, **kw)[0]
            monkeypatch.delenv("EAMG_GROUP_MB", raising=False)
            E.eamg_profile_enable(hier.h, True)
            assert torch.equal(hier.solve_batch(B, **kw)[0], X)
            names[key] = [k["name"] for k in E.eamg_profile_read(hier.h)]
            E.eamg_profile_enable(hier.h, False)
            if key == "groups":
                X0 = X
        assert any(n.endswith(" grouped") for n in names["groups"]), names
        assert not any(n.endswith(" grouped") for n in names["none"]), names
        assert float(((X - X0).norm(dim=1) / X0.norm(dim=1)).max()) <= tol
    h.close()
    ref.close()
