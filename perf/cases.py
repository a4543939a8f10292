"""Performance cases: the calls a program makes on this library, over the sizes it makes them at.

Each case is one call (or the few calls a program always makes together) through the package's
public entry points: equilibrium solves, differentiable solves, interior-point runs in two and
three dimensions, the SIMP variant, the optimality-criteria update loop, and the bare operators.
Grids are the cantilevers of the paper's examples and of the repository's workload table, with odd
coarse grids among them; densities are the random fields that the workloads use."""
import math
import random

import numpy as np
import torch

from paper_1606_06201_amd import Solver, inputs, solve_K

DEV = "cuda:0"

# nx, ny, nz: elements (nz = 0: two dimensions); fp32: precision of the V-cycle (the recurrences
# are always 64 bits); rtol: relative residual of the solves; steps: Newton steps or outer updates.


def listed():
    return [
        # one equilibrium solve on the smallest workload grid: a few launches' worth of work, all latency
        dict(name="solve_64x32", kind="solve", nx=64, ny=32, nz=0, levels=4, fp32=True, rtol=1e-8),
        # an odd coarse grid (9 x 5) in plain 64 bits: what a caller who wants no FP32 anywhere runs
        dict(name="solve_288x160_fp64", kind="solve", nx=288, ny=160, nz=0, levels=6, fp32=False, rtol=1e-8),
        # the ordinary solve: a random-field design at 1024 x 512
        dict(name="solve_1024x512", kind="solve", nx=1024, ny=512, nz=0, levels=7, fp32=True, rtol=1e-8),
        # the largest grid of the workload table (4.2 million unknowns)
        dict(name="solve_2048x1024", kind="solve", nx=2048, ny=1024, nz=0, levels=6, fp32=True, rtol=1e-8),
        # an adjoint gradient: forward solve, backward solve and sensitivities through autograd
        dict(name="adjoint_512x256", kind="adjoint", nx=512, ny=256, nz=0, levels=6, fp32=True, rtol=1e-8),
        # the start and first Newton steps of the interior-point run on the small workload grid
        dict(name="ip_64x32", kind="ip", nx=64, ny=32, nz=0, levels=4, fp32=True, rtol=1e-10, steps=5),
        # the paper's inexact preset (residual 1e-2) on its problem 427, in 64 bits as the tables are run
        dict(name="ip_paper_256x128_fp64", kind="ip", nx=256, ny=128, nz=0, levels=7, fp32=False, rtol=1e-2, steps=6),
        # the three-dimensional interior-point workload, first steps
        dict(name="ip_128x64x64", kind="ip", nx=128, ny=64, nz=64, levels=5, fp32=True, rtol=1e-10, steps=5),
        # a small three-dimensional interior-point run on an odd coarse grid, in 64 bits
        dict(name="ip_40x24x16_fp64", kind="ip", nx=40, ny=24, nz=16, levels=4, fp32=False, rtol=1e-8, steps=4),
        # the SIMP interior-point method (Example 4 of the paper, problem 425)
        dict(name="simp_ip_64x32_fp64", kind="simp_ip", nx=64, ny=32, nz=0, levels=5, fp32=False, rtol=1e-2, steps=3),
        # averaged optimality criteria on problem 426: the loop that the paper's tables compare with
        dict(name="oc_128x64_fp64", kind="oc", nx=128, ny=64, nz=0, levels=6, fp32=False, rtol=1e-4, steps=3),
        # the bare operators of a program with its own outer method: K v, sensitivities, filtered gradient
        dict(name="operators_96x48x40", kind="operators", nx=96, ny=48, nz=40, levels=3, fp32=True, rtol=0.0),
    ]


def draw(rng: random.Random):
    """One more case of the same ranges: a kind, an odd or even coarse grid refined to a size between
    the smallest and the largest that the kind is used at."""
    kind = rng.choice(["solve", "solve", "adjoint", "ip", "ip", "ip3", "solve3", "simp_ip", "oc", "operators"])
    three = kind in ("ip3", "solve3") or (kind == "operators" and rng.random() < 0.6)
    top = {"solve": 1.5e6, "adjoint": 4e5, "ip": 6e4, "ip3": 2.5e5, "solve3": 2.5e5, "simp_ip": 1e4, "oc": 4e4, "operators": 4e5}[kind]
    m = math.exp(rng.uniform(math.log(1000.0), math.log(top)))       # about this many elements
    if three:
        a = (m / 2.0) ** (1.0 / 3.0)
        levels = max(2, int(math.log2(a / 3.0)) + 1 if a > 6 else 2)
        f = 2 ** (levels - 1)
        ny, nz = (max(2, round(a * rng.uniform(0.8, 1.25) / f)) * f for _ in range(2))
        nx = max(3, round(2 * a / f) + rng.choice((0, 1))) * f
    else:
        a = math.sqrt(m / 2.0)
        levels = max(2, int(math.log2(a / rng.uniform(2.0, 12.0))) + 1 if a > 12 else 2)
        f = 2 ** (levels - 1)
        ny, nz = max(2, round(a * rng.uniform(0.7, 1.4) / f)) * f, 0
        nx = max(3, round(m / ny / f) + rng.choice((0, 1))) * f
    # the paper's loose tolerances are used in plain 64 bits; the FP32 V-cycle with tight ones
    fp32 = kind not in ("simp_ip", "oc") and rng.random() < 0.6
    tight = (1e-10,) if kind in ("ip", "ip3", "solve3") else (1e-8, 1e-10)
    rtol = {"simp_ip": 1e-2, "oc": 1e-4, "operators": 0.0}.get(kind, rng.choice(tight if fp32 else (1e-6, 1e-8)))
    case = dict(kind=kind.rstrip("3"), nx=nx, ny=ny, nz=nz, levels=levels, fp32=fp32, rtol=rtol)
    if kind in ("ip", "ip3", "simp_ip", "oc"):
        case["steps"] = rng.randint(2, 4)
    return case


def _nel(case):
    return (case["nx"], case["ny"], case["nz"]) if case["nz"] else (case["nx"], case["ny"])


def _loads(nel, rng):
    """Downward loads on the edge (face) opposite the clamped one, near its middle."""
    if len(nel) == 2:
        nx, ny = nel
        j = ny // 2 + int(rng.integers(-(ny // 8), ny // 8 + 1))
        a = float(rng.uniform(0.8, 1.25))
        return [((nx, j - 1), 1, -0.5 * a), ((nx, j), 1, -a), ((nx, j + 1), 1, -0.5 * a)]
    nx, ny, nz = nel
    out = []
    j0, k0 = ny // 2 + int(rng.integers(-1, 2)), nz // 2 + int(rng.integers(-1, 2))
    for k in range(max(0, k0 - 2), min(nz, k0 + 2)):
        for j in range(max(0, j0 - 2), min(ny, j0 + 2)):
            out.append(((nx, j, k), 1, float(-rng.uniform(0.5, 1.5) / 16.0)))
    return out


def _host_inputs(case, seed):
    """Densities, a load and two fields over the unknowns, made from the seed alone."""
    nel = _nel(case)
    rng = np.random.default_rng(seed)
    m = int(np.prod(nel))
    nslots = len(nel) * int(np.prod([n + 1 for n in nel]))
    d = dict(loads=_loads(nel, rng))
    if case["kind"] == "solve" or case["kind"] == "operators":
        corr = max(2.0, min(16.0, min(nel) / 8.0))
        d["x"] = inputs.density_logistic(nel, seed=int(rng.integers(1 << 30)), corr_len=corr)
    elif case["kind"] == "adjoint":
        d["x"] = inputs.density_uniform(nel, seed=int(rng.integers(1 << 30)))
    else:
        d["x"] = np.full(m, 1.0)
    if case["kind"] in ("adjoint", "operators"):
        d["v"] = rng.standard_normal(nslots)
    if case["kind"] == "operators":
        d["w"] = rng.standard_normal(nslots)
    return d


def prepare(case, seed):
    nel = _nel(case)
    h = _host_inputs(case, seed)
    s = Solver(nel, case["levels"], fp32=case["fp32"], device=DEV)
    st = dict(case=case, s=s, f=s.load_vector(h["loads"]), x=torch.from_numpy(h["x"]).to(DEV))
    for k in ("v", "w"):
        if k in h:
            st[k] = torch.from_numpy(h[k]).to(DEV)
    kind = case["kind"]
    if kind == "ip":
        # the workload's exact settings, or the paper's inexact preset
        three = len(nel) == 3
        st["params"] = (s.ip_params_paper(float(s.m)) if case["rtol"] == 1e-2 else
                        s.ip_params((0.3 if three else 0.5) * s.m, 1.0, pcg_rtol=case["rtol"]))
        st["params"].max_newton = case["steps"]
    elif kind == "simp_ip":
        st["params"] = s.ip_params_paper(float(s.m), xbar=3.0)
        st["params"].max_newton = case["steps"]
    elif kind == "operators":
        s.set_density(st["x"])
    return st


def run(state):
    case, s, f = state["case"], state["s"], state["f"]
    kind = case["kind"]
    if kind == "solve":
        s.set_density(state["x"])
        u, info = s.pcg(f, rtol=case["rtol"])
        return {"u": u, "compliance": info["bu"]}
    if kind == "adjoint":
        x = state["x"].requires_grad_(True)
        u = solve_K(x, f, s, rtol=case["rtol"])
        gx, = torch.autograd.grad(u, x, state["v"])
        return {"u": u.detach(), "gx": gx}
    if kind == "ip":
        st, log = s.ip_run(f, state["params"])
        return {"state": st, "compliance": log["steps"][-1]["compliance"]}
    if kind == "simp_ip":
        st, log = s.ip_run(f, state["params"], cg_tol_factor=0.5, simp=(2.0, 3.0))
        return {"state": st, "compliance": log["steps"][-1]["compliance"]}
    if kind == "oc":
        x, u, log = s.oc_run(f, state["x"], float(s.m), 2.0, variant="aoc", cg_tol=case["rtol"], max_outer=case["steps"])
        return {"x": x, "u": u, "compliance": log["compliance"]}
    y = s.apply_K(state["v"])
    g = s.element_sens(state["w"], state["v"], -1.0)
    return {"y": y, "g": g, "filtered": s.filter(g, 2.0, transpose=True)}


def work(case):
    """What a pass cannot do without: each vector of a PCG step read or written once where a step
    needs it (direction, operator, update: 96 bytes an unknown in two dimensions; the V-cycle reads
    its right-hand side and writes its result on every level), times the steps that these systems
    take; the bare operators' own inputs and outputs."""
    nel = _nel(case)
    dim = len(nel)
    m = float(np.prod(nel))
    n = dim * float(np.prod([k + 1 for k in nel]))
    el = (2.0 * (dim * 2 ** dim) ** 2) * m                          # one operator apply
    if case["kind"] == "operators":
        return {"bytes": 8.0 * (2 * n + m) + 8.0 * (2 * n + m) + 16.0 * m, "flops": 2.0 * el}
    its = {"solve": 25.0 if dim == 2 else 18.0, "adjoint": 28.0, "ip": 14.0, "simp_ip": 14.0, "oc": 8.0}[case["kind"]]
    if case["rtol"] == 1e-2 and case["kind"] == "ip":
        its = 4.0
    its *= {"ip": case.get("steps", 0) * 0.6 + 1, "simp_ip": case.get("steps", 0) + 1, "oc": 2 * case.get("steps", 0) + 1}.get(case["kind"], 1)
    w = 4.0 if case["fp32"] else 8.0
    cyc = 4.0 / 3.0 if dim == 2 else 8.0 / 7.0                       # all levels against the finest
    per = 8.0 * (4 * n + 3 * n) + 8.0 * m + cyc * (2 * w * n + w * m)
    return {"bytes": its * per, "flops": its * el * (1.0 + 5.0 * cyc)}


def _element_matrix(dim, E=1.0, nu=0.3):
    """Q1 element stiffness of the unit square (plane stress) or cube, two Gauss points per axis."""
    off = [(0, 0, 0), (1, 0, 0), (1, 1, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1)][: 2 ** dim]
    mu = E / (2 * (1 + nu))
    lam = E * nu / (1 - nu * nu) if dim == 2 else E * nu / ((1 + nu) * (1 - 2 * nu))
    g = 0.5 / math.sqrt(3.0)
    nn = len(off)
    K = np.zeros((nn, dim, nn, dim))
    for p in np.ndindex(*(2,) * dim):
        xi = [0.5 - g if q == 0 else 0.5 + g for q in p]
        G = np.ones((nn, dim))
        for a in range(nn):
            for i in range(dim):
                for e in range(dim):
                    G[a, i] *= (1.0 if off[a][e] else -1.0) if e == i else (xi[e] if off[a][e] else 1 - xi[e])
        K += (lam * np.einsum("ai,bj->aibj", G, G) + mu * np.einsum("aj,bi->aibj", G, G)
              + mu * np.einsum("ak,bk,ij->aibj", G, G, np.eye(dim))) / 2 ** dim
    return K.reshape(nn * dim, nn * dim), off


def _element_slots(nel):
    dim = len(nel)
    _, off = _element_matrix(dim)
    nx, ny = nel[:2]
    nz = nel[2] if dim == 3 else 1
    k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    cols = []
    for o in off:
        q = ((k + o[2]) * (ny + 1) + (j + o[1])) * (nx + 1) + i + o[0]
        cols += [dim * q.ravel() + c for c in range(dim)]
    return np.stack(cols, 1)


def exact(case, seed):
    """The same outputs in 64 bits with plain numpy and torch: the operators at any size, a solve
    where a dense factorization is quick."""
    nel = _nel(case)
    dim = len(nel)
    if case["kind"] not in ("operators", "solve"):
        return None
    h = _host_inputs(case, seed)
    K0, _ = _element_matrix(dim)
    e = _element_slots(nel)
    n = dim * int(np.prod([k + 1 for k in nel]))
    free = (np.arange(n) // dim) % (nel[0] + 1) != 0
    if case["kind"] == "operators":
        v, w = np.where(free, h["v"], 0.0), np.where(free, h["w"], 0.0)
        ye = (v[e] @ K0) * h["x"][:, None]
        y = np.where(free, np.bincount(e.ravel(), ye.ravel(), n), 0.0)
        g = -np.einsum("ma,ma->m", w[e] @ K0, v[e])
        shape = nel[::-1]
        return {"y": y, "g": g, "filtered": _filter_transposed(g.reshape(shape), 2.0).ravel()}
    if n > 5000:
        return None
    K = np.zeros((n, n))
    for a in range(e.shape[1]):
        for b in range(e.shape[1]):
            np.add.at(K, (e[:, a], e[:, b]), h["x"] * K0[a, b])
    f = np.zeros(n)
    strides = (1, nel[0] + 1, (nel[0] + 1) * (nel[1] + 1))
    for at, c, val in h["loads"]:
        f[dim * sum(p * s for p, s in zip(at, strides)) + c] += val
    f[~free] = 0.0
    K[~free, :] = 0.0
    K[:, ~free] = 0.0
    K[~free, ~free] = 1.0
    u = torch.linalg.solve(torch.from_numpy(K), torch.from_numpy(f)).numpy()
    return {"u": u, "compliance": float(f @ u)}


def _filter_transposed(g, rmin):
    """W' g of the density filter: weights max(0, rmin - Manhattan distance), columns scaled to one."""
    r = int(math.ceil(rmin)) - 1

    def spread(a):
        out = np.zeros_like(a)
        for o in np.ndindex(*(2 * r + 1,) * a.ndim):
            o = [q - r for q in o]
            wt = rmin - sum(abs(q) for q in o)
            if wt <= 0:
                continue
            dst = tuple(slice(max(0, -q), min(s, s - q)) for q, s in zip(o, a.shape))
            src = tuple(slice(max(0, q), min(s, s + q)) for q, s in zip(o, a.shape))
            out[dst] += wt * a[src]
        return out

    return spread(g) / spread(np.ones_like(g))
