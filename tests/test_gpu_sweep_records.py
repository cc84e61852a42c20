"""Bytes and names of the sweeps in the profiler's records and in the traffic model: what the colours of the
matrix need by the documented counts (every block and index once, gathered entries once per launch, row
data), whether the colours run one by one or as groups, and a group's launches under a name of their own.
The counts are formed here from the exported levels; they are whole numbers below 2^53, so equality holds
up to the rounding of a few additions (1e-12)."""
import re

import numpy as np
import pytest

import paper_2011_13325_amd as E
from gen import make_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "elasticity": dict(n=19, ny=17, nz=18, nu=0.3),
    "poisson": dict(n=41, ny=37, nz=39, kind="poisson", clamp="all"),
}
SWEEP = re.compile(r"L(\d+) c(\d+)(?:-(\d+))? k_gs_color<\w+, \d+, (true|false)>( grouped)?$")


def _sweep_bytes(lv, vs):
    """{(forward, colour): bytes} of one level."""
    n, bs, rp, col, color = lv["info"]["n"], lv["info"]["bs"], lv["A_rowptr"], lv["A_col"], lv["color"]
    rows = np.repeat(np.arange(n), np.diff(rp))
    left = color[col] <= color[rows]   # with the diagonal: rows of a colour are not coupled
    out = {}
    for c in range(int(color.max()) + 1):
        for fwd in (True, False):
            q = (color[rows] == c) & (left if fwd else True)
            out[fwd, c] = (q.sum() * (bs * bs * vs + 4) + np.unique(col[q]).size * bs * vs
                           + (color == c).sum() * (8 + bs * bs * vs + (3 if fwd else 2) * bs * vs))
    return out


def _vcycle_bytes(levels, vs):
    total = 0
    for lv in levels[:-1]:
        n, bs, kc = (lv["info"][f] for f in ("n", "bs", "k_coarse"))
        rp, col, color = lv["A_rowptr"], lv["A_col"], lv["color"]
        rows = np.repeat(np.arange(n), np.diff(rp))
        right = color[col] > color[rows]
        nc, nP = int(lv["agg"].max()) + 1, lv["P_col"].size
        blk = nP * (bs * kc * vs + 4)
        total += sum(_sweep_bytes(lv, vs).values())
        total += right.sum() * (bs * bs * vs + 4) + np.unique(col[right]).size * bs * vs + n * (8 + 2 * bs * vs)
        total += blk + (np.diff(lv["P_rowptr"]) > 0).sum() * bs * vs + 4 * (nc + 1) + nc * kc * vs
        total += blk + np.unique(lv["P_col"]).size * kc * vs + 4 * (n + 1) + 2 * n * bs * vs
    nL = levels[-1]["info"]["n"] * levels[-1]["info"]["bs"]
    return total + nL * nL * 8 + 2 * nL * vs


@pytest.mark.parametrize("name", list(CASES))
def test_sweep_bytes_are_those_of_the_colours(name):
    p = make_problem(**CASES[name])
    h = E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                    E.eamg_default_setup_params(vcycle_fp32=1))
    levels = [h.export(l) for l in range(h.stats()["n_levels"])]
    for prec, vs in ((E.EAMG_PRECOND_VCYCLE, 8), (E.EAMG_PRECOND_VCYCLE_FP32, 4)):
        assert E.eamg_traffic_model(h.h, prec)[0] == pytest.approx(_vcycle_bytes(levels, vs), rel=1e-12)
    r = torch.ones(p.n_dofs, dtype=torch.float64, device="cuda")
    z = torch.empty_like(r)
    E.eamg_profile_enable(h.h, 3)
    E.eamg_vcycle(h.h, r, z)
    ks = E.eamg_profile_read(h.h, 4096)
    stages = [SWEEP.match(k["name"]) for k in ks]
    E.eamg_profile_enable(h.h, 2)
    E.eamg_vcycle(h.h, r, z)
    runs = {k["name"]: k for k in E.eamg_profile_read(h.h, 4096)}
    E.eamg_profile_enable(h.h, False)
    groups = 0
    for l, lv in enumerate(levels[:-1]):
        want = _sweep_bytes(lv, 8)
        nc = int(lv["color"].max()) + 1
        for fwd in (True, False):
            seen, grouped = [], 0.0
            for k, m in zip(ks, stages):
                if not m or int(m[1]) != l or (m[4] == "true") != fwd:
                    continue
                c0, c1 = int(m[2]), int(m[3] or m[2])
                assert (c1 > c0) == bool(m[5]), k["name"]
                assert k["launches"] == (1 if not m[5] or (fwd and c0 == 0) else 2), k
                bytes_ = sum(want[fwd, c] for c in range(c0, c1 + 1))
                assert k["bytes"] == pytest.approx(bytes_, rel=1e-12), k
                seen += range(c0, c1 + 1)
                grouped += bytes_ if m[5] else 0.0
            assert sorted(seen) == list(range(nc)), (l, fwd, seen)
            groups += grouped > 0
            base = f"L{l} k_gs_color<double, {lv['info']['bs']}, {'true' if fwd else 'false'}>"
            total = sum(want[fwd, c] for c in range(nc))
            one_by_one = runs[base]["bytes"] if base in runs else 0.0
            as_groups = runs[base + " grouped"]["bytes"] if base + " grouped" in runs else 0.0
            assert as_groups == pytest.approx(grouped, rel=1e-12)
            assert one_by_one + as_groups == pytest.approx(total, rel=1e-12)
    print(f"\n[{name}] {len(levels)} levels, sweeps with groups {groups}", flush=True)
    assert groups
    h.close()
