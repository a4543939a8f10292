"""Finest 3D level in one pass (element products and node sums, marching along z):
grids at the edges of its 32 x 8 node columns and of its plane chunks, against the
oracle and the gather form (IPMG_NO_ELEM_FINE3).  Bounds as for the operator and
V-cycle parity tests."""
import numpy as np
import pytest

from oracle import fem, mg
from tests.gpu_util import T, N, relerr, grid_and_k0, tip_load
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu

# columns 1..32 in one tile, one and two past it; rows 7, 8 and 9; one to eleven planes
GRIDS = [((2, 2, 2), 1), ((32, 6, 4), 2), ((34, 8, 2), 2), ((66, 10, 10), 2)]


@pytest.mark.parametrize("nel,levels", GRIDS)
@pytest.mark.parametrize("fp32", [False, True])
def test_operators_and_vcycle(nel, levels, fp32, monkeypatch):
    from paper_1606_06201_amd import Solver
    prob = _problem(nel)
    g = prob.grid
    st, u_slots = _state(prob)
    Z, _, _ = prob.z_system(st)
    free = g.free_to_slot()
    monkeypatch.setenv("IPMG_NO_TAIL", "1")           # the finest level's own passes on small grids too
    s = Solver(nel, levels, fp32=fp32)
    s.ip_prepare(T(prob.f_slots), s.ip_params(prob.V, prob.xbar), _gpu_state(s, st, u_slots))
    v = np.random.default_rng(3).standard_normal(g.nslots + 1)
    _, K0 = grid_and_k0(nel)
    y = N(s.apply_K(T(v[:-1])))                        # clamped entries are ignored by contract
    assert relerr(y, fem.apply_free_masked(g, st.x, K0, v[:-1])) < 1e-13
    assert np.all(y[g.clamped_mask()] == 0)
    v[:-1][g.clamped_mask()] = 0
    vf = np.concatenate([v[:-1][free], v[-1:]])
    y = N(s.apply_Z(T(v)))
    assert relerr(np.concatenate([y[:-1][free], y[-1:]]), Z @ vf) < 1e-12
    for op, H, tol in ((1, mg.Hierarchy(g, Z, levels, augmented=True), 1e-9),
                       (0, mg.kstiffness_hierarchy(g, st.x, K0, levels), 1e-11)):
        s.mg_setup(op)
        ev = np.linalg.eigvalsh(H.A[0].toarray())
        tol = max(tol, np.finfo(float).eps * ev[-1] / ev[0])
        if levels > 1:
            assert abs(s.level_damping(1)[1] - H.rho[1]) <= (1e-4 if fp32 else 1e-9) * H.rho[1]
        z = N(s.vcycle(T(v if op else v[:-1]), op=op))
        ref = mg.vcycle(H, vf if op else v[:-1][free])
        got = np.concatenate([z[:-1][free], z[-1:]]) if op else z[free]
        assert relerr(got, ref) < (2e-4 if fp32 else tol)
        assert np.all((z[:-1] if op else z)[g.clamped_mask()] == 0)


@pytest.mark.parametrize("nel,levels", GRIDS[1:])
@pytest.mark.parametrize("fp32", [False, True])
def test_pcg_direction(nel, levels, fp32, monkeypatch):
    # the PCG direction formed inside the pass: the same steps as with the gather form
    # (solutions to the tolerance of the solve, counts within one)
    from paper_1606_06201_amd import Solver
    g, K0 = grid_and_k0(nel)
    x = np.random.default_rng(5).uniform(0.1, 1.0, g.m)
    f = np.zeros(g.nslots)
    f[3 * int(g.node_index(nel[0], nel[1] // 2, nel[2] // 2)) + 1] = -1.0
    out = []
    for off in ("0", "1"):
        monkeypatch.setenv("IPMG_NO_ELEM_FINE3", off)
        s = Solver(nel, levels, fp32=fp32)
        s.set_density(T(x))
        u, info = s.pcg(T(f), rtol=1e-10)
        assert info["true_relres"] <= 1e-10
        out.append((N(u), info["iters"]))
    assert abs(out[0][1] - out[1][1]) <= 1
    assert relerr(out[0][0], out[1][0]) < 1e-8
