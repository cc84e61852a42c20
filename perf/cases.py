"""Timed workloads of the AMG-PCG library, from the smallest calls to the 128^3 headline.

Each case is one call a program makes through the package's public entry points: a solve with a
hierarchy that the program keeps (one mesh, many right-hand sides), a block of load cases, many
meshes solved together, a bare V-cycle (the preconditioner of a caller's own Krylov method), a
one-shot setup and solve, and one training gradient of the edge network.  ``prepare`` makes the
right-hand sides from the seed and keeps the hierarchy of a mesh from one call to the next, as
such a program does; the hierarchies kept are bounded (``_KEEP``).
"""
import collections
import math

import numpy as np
import torch

import paper_2011_13325_amd as E
from gen import make_problem

# Setup parameters.  "default": the library's defaults (the paper's row caps, every level's sweeps
# sparse).  "tuned": the settings of the cube workloads in bench.py (row caps 6/4/4, sigma 18,
# dense V-cycle tail), with the launch-shape autotuner.  "multi": bench.py's settings of the small
# meshes solved together (row caps 6/4/3, sigma 20).
SETTINGS = {
    "default": dict(vcycle_fp32=1),
    "tuned": dict(vcycle_fp32=1, dense_tail_dofs=16384, cap_std_l0=6, cap_std=4, cap_aux=4, sigma=18.0),
    "multi": dict(vcycle_fp32=1, dense_tail_dofs=16384, cap_std_l0=6, cap_std=4, cap_aux=3, sigma=20.0),
}
PRECOND = {"f64": E.EAMG_PRECOND_VCYCLE, "f32": E.EAMG_PRECOND_VCYCLE_FP32}


def _solve(name, nx, ny, nz, settings, precision, kind="elasticity", nu=0.3):
    return dict(name=name, what="solve", nx=nx, ny=ny, nz=nz, kind=kind, nu=nu, settings=settings,
                precision=precision)


def listed():
    return [
        # the smallest call: a toy mesh, two levels, every launch a few rows; latency alone counts
        _solve("solve 7^3 f64", 7, 7, 7, "default", "f64"),
        # a small model with the library's defaults (the bench's CPU-comparison cube)
        _solve("solve 17^3 f64", 17, 17, 17, "default", "f64"),
        # scalar problem (1x1 blocks on every level), a box of odd sides, defaults but for the size
        _solve("poisson 65x57x71 f64", 65, 57, 71, "default", "f64", kind="poisson"),
        # an ordinary elasticity model, all in FP64
        _solve("solve 64^3 f64", 64, 64, 64, "tuned", "f64"),
        # the same with the FP32 V-cycle, as a production program would run it
        _solve("solve 64^3 f32", 64, 64, 64, "tuned", "f32"),
        # the largest: the bench's headline, nearly incompressible, 6.3 M dofs
        _solve("solve 128^3 f32", 128, 128, 128, "tuned", "f32", nu=0.45),
        # many load cases on one mesh (block panels)
        dict(name="batch 64^3 x32 f32", what="batch", nx=64, ny=64, nz=64, nu=0.3, nrhs=32,
             settings="tuned", precision="f32"),
        # a few load cases on a ragged box, all in FP64: a panel that is not full
        dict(name="batch 37x29x33 x7 f64", what="batch", nx=37, ny=29, nz=33, nu=0.35, nrhs=7,
             settings="tuned", precision="f64"),
        # independent meshes of uneven size solved together (the bench's 16 cubes of 8^3..48^3)
        dict(name="fused 16 meshes f32", what="fused", count=16, lo=8, hi=48, mesh_seed=4,
             precision="f32"),
        # the preconditioner alone, inside a caller's own Krylov method; ragged box
        dict(name="vcycle 41x23x31 f64", what="vcycle", nx=41, ny=23, nz=31, nu=0.35,
             settings="tuned", precision="f64"),
        # one mesh, one load: setup from host arrays and the solve; stiff inclusions (E = 1e4)
        dict(name="setup+solve 21^3 f32", what="oneshot", nx=21, inclusions=4, precision="f32"),
        # one training gradient of the edge network on a pass graph of a mid-size mesh
        dict(name="edge network 60001", what="gnn", pairs=60001, nodes=16000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["solve", "solve", "solve", "batch", "fused", "vcycle", "oneshot", "gnn"])
    side = lambda lo, hi: dict(zip(("nx", "ny", "nz"), (_log_int(rng, lo, hi) for _ in range(3))))
    # the tuned sigma is for nu >= 0.3; below, meshes take the settings of the uneven ones
    nu = round(rng.uniform(0.2, 0.45), 4)
    settings = "tuned" if nu >= 0.3 else "multi"
    precision = rng.choice(["f64", "f32"])
    if what == "solve":
        if rng.random() < 0.25:
            return dict(what="solve", kind="poisson", nu=0.3, settings="default", precision="f64",
                        **side(9, 90))
        n = _log_int(rng, 6, 80)
        lo, hi = max(5, int(0.8 * n)), int(1.2 * n) + 1
        return dict(what="solve", kind="elasticity", nu=nu, precision=precision,
                    settings="default" if n < 30 and rng.random() < 0.5 else settings, **side(lo, hi))
    if what == "batch":
        return dict(what="batch", nu=nu, nrhs=_log_int(rng, 2, 64), settings=settings,
                    precision=precision, **side(12, 52))
    if what == "fused":
        lo = rng.randint(6, 12)
        return dict(what="fused", count=rng.randint(2, 16), lo=lo, hi=rng.randint(lo + 4, 36),
                    mesh_seed=rng.randint(5, 1000), precision=precision)
    if what == "vcycle":
        return dict(what="vcycle", nu=nu, settings=settings, precision="f64", **side(9, 56))
    if what == "oneshot":
        return dict(what="oneshot", nx=rng.randint(8, 21), inclusions=rng.randint(1, 5), precision=precision)
    m = _log_int(rng, 1000, 100000)
    return dict(what="gnn", pairs=m, nodes=max(4, m // rng.randint(2, 6)))


# ---- hierarchies kept from call to call ------------------------------------------------------
_KEEP = 2
_kept = collections.OrderedDict()


def _keep(key, make):
    if key in _kept:
        _kept.move_to_end(key)
    else:
        while len(_kept) >= _KEEP:
            _kept.popitem(last=False)   # closed with its last state
        _kept[key] = make()
    return _kept[key]


def _problem(case):
    kw = dict(kind=case.get("kind", "elasticity"))
    if case.get("kind") == "poisson":
        kw["clamp"] = "all"
    return make_problem(case["nx"], ny=case["ny"], nz=case["nz"], nu=case["nu"], **kw)


def _setup(p, params):
    return E.Hierarchy(p.dim, p.coords, p.row_ptr, p.col_idx, p.vals, p.dirichlet,
                       E.eamg_default_setup_params(**params))


def _hierarchy(case):
    """(problem's free-dof mask on the GPU, hierarchy) of a case's mesh."""
    width = 0
    if case["what"] == "batch":
        width = 1 << min(6, max(0, case["nrhs"] - 1).bit_length())

    def make():
        p = _problem(case)
        h = _setup(p, SETTINGS[case["settings"]])
        if case["settings"] != "default":
            E.eamg_autotune(h.h, panel_width=width)
        free = np.repeat(p.dirichlet == 0, p.dim)
        return torch.tensor(free, device="cuda"), h

    key = ("mesh", case["nx"], case["ny"], case["nz"], case["nu"], case.get("kind"), case["settings"], width)
    return _keep(key, make)


def _meshes(case):
    """Sides and Poisson ratios of a fused case's cubes."""
    rng = np.random.default_rng(case["mesh_seed"])
    sides = rng.integers(case["lo"], case["hi"] + 1, size=case["count"])
    return [int(s) for s in sides], [float(v) for v in rng.uniform(0.2, 0.45, size=case["count"])]


def _fused(case):
    def make():
        parts, free = [], []
        for n, nu in zip(*_meshes(case)):
            p = make_problem(n, nu=nu)
            parts.append(_setup(p, SETTINGS["multi"]))
            free.append(torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda"))
        f = E.Fused(parts, dense_tail_dofs=4096)
        E.eamg_autotune(f.h, 0)
        return free, f

    return _keep(("fused", case["count"], case["lo"], case["hi"], case["mesh_seed"]), make)


def _loads(free, seed, *lead):
    """Seeded load vectors, uniform in [-1, 1], zero at the clamped dofs."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    b = torch.rand(*lead, free.numel(), dtype=torch.float64, device="cuda", generator=g) * 2 - 1
    return b * free


def _pass_graph(case, seed):
    """A candidate-pair graph with features, labels and weights like a recorded matching pass."""
    rng = np.random.default_rng(seed)
    m, n = case["pairs"], case["nodes"]
    X = rng.standard_normal((m, E.GNN_FEATURES)).astype(np.float32)
    u = rng.integers(0, n, size=m)
    v = (u + rng.integers(1, min(n, 64), size=m)) % n
    edges = np.sort(np.stack([u, v], axis=1), axis=1).astype(np.int32)
    y = (rng.random(m) < 0.4).astype(np.float32)
    w = (rng.random(m) < 0.7).astype(np.float32)
    parts = [rng.uniform(-1, 1, 64 * 12) * math.sqrt(6 / 12), rng.uniform(-0.1, 0.1, 64),
             rng.uniform(-1, 1, 64 * 64) * math.sqrt(6 / 64), rng.uniform(-1, 1, 64 * 64) * math.sqrt(6 / 64),
             rng.uniform(-0.1, 0.1, 64), rng.uniform(-1, 1, 64) * math.sqrt(6 / 64), [0.05]]
    return X, edges, n, y, w, np.concatenate(parts).astype(np.float32)


def _oneshot_problem(case, seed):
    # the inclusions' places too are drawn from the seed: every setup is a new one
    return make_problem(case["nx"], inclusions=case["inclusions"], geometry_seed=seed, seed=seed)


def prepare(case, seed):
    what = case["what"]
    if what in ("solve", "batch", "vcycle"):
        free, h = _hierarchy(case)
        lead = (case["nrhs"],) if what == "batch" else ()
        return case, h, _loads(free, seed, *lead)
    if what == "fused":
        free, f = _fused(case)
        return case, f, [_loads(fr, seed * 64 + i) for i, fr in enumerate(free)]
    if what == "oneshot":
        p = _oneshot_problem(case, seed)
        return case, p, torch.tensor(p.b, device="cuda")
    X, edges, n, y, w, params = _pass_graph(case, seed)
    return case, E.EdgeNet(params), (X, edges, n, y, w)


def run(state):
    case, h, b = state
    what = case["what"]
    if what == "solve":
        x, info = h.solve(b, precond=PRECOND[case["precision"]])
        return x, info["iterations"]
    if what == "batch":
        X, _, infos = h.solve_batch(b, precond=PRECOND[case["precision"]])
        return X, np.array([i["iterations"] for i in infos])
    if what == "fused":
        xs, _, infos = h.solve(b, precond=PRECOND[case["precision"]])
        return xs, np.array([i["iterations"] for i in infos])
    if what == "vcycle":
        z = torch.empty_like(b)
        E.eamg_vcycle(h.h, b, z, PRECOND[case["precision"]])
        return z
    if what == "oneshot":
        hier = _setup(h, SETTINGS["multi"])
        x, info = hier.solve(b, precond=PRECOND[case["precision"]])
        sizes = np.array(hier.stats()["nnzb"])
        hier.close()
        return x, info["iterations"], sizes
    return h.loss_grad(*b)


# ---- the work a pass cannot do without -------------------------------------------------------
def _fine_blocks(nx, ny, nz):
    """Blocks of the finest matrix of a box: each vertex and, twice, each edge of its seven
    directions."""
    edges = 0
    for d in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, 0, 1), (0, 1, 1), (1, 1, 1)):
        edges += (nx - d[0]) * (ny - d[1]) * (nz - d[2])
    return nx * ny * nz + 2 * edges


# Operator complexity (entries of all levels over those of the finest) by settings, as measured.
_COMPLEXITY = {"default": 8.9, "tuned": 7.2, "multi": 5.7, "poisson": 2.3}


def _iterations(n):
    """Typical PCG iterations to 1e-8 at a mean side of n vertices."""
    return max(8, round(4 * math.log2(n) - 6))


def _cycle_entries(nx, ny, nz, dim, complexity):
    """Matrix entries a V-cycle reads: every level's matrix before and after its coarse
    correction, and the transfers (about a third of a matrix, each way)."""
    return _fine_blocks(nx, ny, nz) * dim * dim * complexity * 2.6


def _solve_work(nx, ny, nz, dim, complexity, precision, nrhs=1):
    size = 4 if precision == "f32" else 8
    a0 = _fine_blocks(nx, ny, nz) * dim * dim
    cyc = _cycle_entries(nx, ny, nz, dim, complexity)
    its = _iterations((nx * ny * nz) ** (1 / 3))
    vec = nx * ny * nz * dim * 8 * 10 * nrhs   # CG's vectors: ten reads and writes an iteration
    return dict(bytes=its * (a0 * 8 + cyc * size + vec), flops=its * 2 * (a0 + cyc) * nrhs)


def work(case):
    what = case["what"]
    if what in ("solve", "batch"):
        poisson = case.get("kind") == "poisson"
        return _solve_work(case["nx"], case["ny"], case["nz"], 1 if poisson else 3,
                           _COMPLEXITY["poisson" if poisson else case["settings"]],
                           case["precision"], case.get("nrhs", 1))
    if what == "fused":
        ws = [_solve_work(n, n, n, 3, _COMPLEXITY["multi"], case["precision"]) for n in _meshes(case)[0]]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if what == "vcycle":
        e = _cycle_entries(case["nx"], case["ny"], case["nz"], 3, _COMPLEXITY[case["settings"]])
        return dict(bytes=e * 8, flops=2 * e)
    if what == "oneshot":
        n = case["nx"]
        w = _solve_work(n, n, n, 3, _COMPLEXITY["multi"], case["precision"])
        # the setup reads A, forms each level's P_s and P_s^T A P_s (two block products)
        entries = _fine_blocks(n, n, n) * 9 * _COMPLEXITY["multi"]
        return dict(bytes=w["bytes"] + entries * 8 * 4, flops=w["flops"] + entries * 2 * 24)
    m = case["pairs"]
    return dict(bytes=m * (12 * 4 + 2 * 4 + 2 * 4) + 2 * 4 * E.GNN_PARAMS, flops=3 * 2 * m * 64 * (12 + 64 + 64 + 1))


# ---- 64-bit reference values -----------------------------------------------------------------
def _system(p):
    """The masked system (identity at clamped dofs) as a scalar CSR matrix, and its diagonal."""
    n, dim = p.n_vertices, p.dim
    rp = torch.tensor(p.row_ptr, device="cuda", dtype=torch.int64)
    col = torch.tensor(p.col_idx, device="cuda", dtype=torch.int64)
    val = torch.tensor(p.vals, device="cuda").reshape(-1, dim, dim)
    fixed = torch.tensor(p.dirichlet, device="cuda").bool()
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), rp[1:] - rp[:-1])
    val = val * (~(fixed[row] | fixed[col]))[:, None, None]
    val = val + (fixed[row] & (row == col))[:, None, None] * torch.eye(dim, device="cuda", dtype=torch.float64)
    c = torch.arange(dim, device="cuda")
    i = (row[:, None, None] * dim + c[:, None]).expand_as(val).reshape(-1)
    j = (col[:, None, None] * dim + c).expand_as(val).reshape(-1)
    a = torch.sparse_coo_tensor(torch.stack([i, j]), val.reshape(-1), (n * dim, n * dim))
    at = row == col
    return a.coalesce().to_sparse_csr(), torch.diagonal(val[at], dim1=1, dim2=2).reshape(-1, 1)


def _conjugate_gradients(p, B, rtol=1e-12, limit=20000):
    """Solution of the masked system for each row of B, by diagonally preconditioned CG."""
    a, diag = _system(p)
    b = B.T.contiguous()
    dot = lambda u, v: (u * v).sum(dim=0)
    x, r = torch.zeros_like(b), b.clone()
    z = r / diag
    d, rz, stop = z.clone(), dot(r, z), rtol * dot(b, b).sqrt()
    for k in range(limit):
        q = a @ d
        alpha = rz / dot(d, q).clamp_min(1e-300)
        x += alpha * d
        r -= alpha * q
        z = r / diag
        new = dot(r, z)
        d = z + (new / rz.clamp_min(1e-300)) * d
        rz = new
        if k % 25 == 24 and bool((dot(r, r).sqrt() <= stop).all()):
            break
    return x.T.contiguous()


def _network_reference(X, edges, n, y, w, params):
    """Loss and parameter gradient of the edge network in float64 (weights rounded to bfloat16,
    as the network uses them)."""
    q, at, leaves = torch.tensor(params), 0, []
    for shape, rounded in (((64, 12), True), ((64,), False), ((64, 64), True), ((64, 64), True),
                           ((64,), False), ((64,), True), ((1,), False)):
        k = int(np.prod(shape))
        v = q[at:at + k]
        v = v.to(torch.bfloat16).double() if rounded else v.double()
        leaves.append(v.reshape(shape).clone().requires_grad_())
        at += k
    W1, b1, W2a, W2b, b2, w3, b3 = leaves
    X, u, v = torch.tensor(X).double(), torch.tensor(edges[:, 0]).long(), torch.tensor(edges[:, 1]).long()
    y, w = torch.tensor(y).double(), torch.tensor(w).double()
    h1 = torch.relu(X @ W1.T + b1)
    deg = torch.zeros(n, dtype=torch.float64).index_add(0, u, torch.ones_like(y)).index_add(0, v, torch.ones_like(y))
    mean = torch.zeros(n, 64, dtype=torch.float64).index_add(0, u, h1).index_add(0, v, h1) / deg.clamp_min(1)[:, None]
    h2 = torch.relu(h1 @ W2a.T + (mean[u] + mean[v]) @ W2b.T + b2)
    z = h2 @ w3 + b3
    loss = (w * torch.nn.functional.binary_cross_entropy_with_logits(z, y, reduction="none")).sum() / w.sum()
    loss.backward()
    return float(loss.detach()), torch.cat([t.grad.reshape(-1) for t in leaves]).numpy()


def exact(case, seed):
    what = case["what"]
    if what == "vcycle":
        return None   # the value of the multilevel method itself: no plain formula
    if what == "gnn":
        return _network_reference(*_pass_graph(case, seed))
    if what == "oneshot":
        p = _oneshot_problem(case, seed)
        return _conjugate_gradients(p, torch.tensor(p.b, device="cuda")[None])[0], None, None
    if what == "fused":
        xs = []
        for i, (n, nu) in enumerate(zip(*_meshes(case))):
            p = make_problem(n, nu=nu)
            free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
            xs.append(_conjugate_gradients(p, _loads(free, seed * 64 + i)[None])[0])
        return xs, None
    if case["nx"] * case["ny"] * case["nz"] > 100 ** 3:
        return None   # plain CG takes thousands of steps there
    p = _problem(case)
    free = torch.tensor(np.repeat(p.dirichlet == 0, p.dim), device="cuda")
    if what == "batch":
        return _conjugate_gradients(p, _loads(free, seed, case["nrhs"])), None
    return _conjugate_gradients(p, _loads(free, seed)[None])[0], None
