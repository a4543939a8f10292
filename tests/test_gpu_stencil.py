"""Levels in node-stencil form and the one-workgroup V-cycle of small levels, for K and
for the augmented system Z, against the FP64 oracle.  Bounds as for the V-cycle
parity tests: FP64 1e-11 (K) and 1e-9 (Z, whose rank-one terms raise the condition
number), FP32 2e-4."""
import numpy as np
import pytest

from oracle import fem, mg, pcg as opcg
from tests.gpu_util import T, N, relerr, grid_and_k0, tip_load
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu

# whole hierarchy in the tail (one tile, several, more tiles than waves); the coarsest
# solve outside it (orders 1122 and 1024); the finest level above it, on odd coarse
# grids; 3D with the tail on the lowest level only and on all
GRIDS = [((8, 4), 2), ((16, 8), 3), ((64, 32), 4), ((64, 32), 2), ((62, 30), 2), ((40, 24), 4), ((144, 80), 5),
         ((8, 4, 4), 3), ((12, 8, 4), 2), ((20, 12, 8), 3)]


@pytest.mark.parametrize("nel,levels", GRIDS)
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("tail", [True, False])
def test_vcycle_and_damping(nel, levels, fp32, tail, monkeypatch):
    from paper_1606_06201_amd import Solver
    prob = _problem(nel)
    g = prob.grid
    st, u_slots = _state(prob)
    Z, _, _ = prob.z_system(st)
    free = g.free_to_slot()
    if not tail:
        monkeypatch.setenv("IPMG_NO_TAIL", "1")
    s = Solver(nel, levels, fp32=fp32)
    s.ip_prepare(T(prob.f_slots), s.ip_params(prob.V, prob.xbar), _gpu_state(s, st, u_slots))
    v = np.random.default_rng(3).standard_normal(g.nslots + 1)
    v[:-1][g.clamped_mask()] = 0
    _, K0 = grid_and_k0(nel)
    for op, H, tol in ((1, mg.Hierarchy(g, Z, levels, augmented=True), 1e-9),
                       (0, mg.kstiffness_hierarchy(g, st.x, K0, levels), 1e-11)):
        s.mg_setup(op)
        for k in range(1, levels):
            assert abs(s.level_damping(k)[1] - H.rho[k]) <= (1e-4 if fp32 else 1e-9) * H.rho[k]
        r = v if op else v[:-1]
        z = N(s.vcycle(T(r), op=op))
        ref = mg.vcycle(H, np.concatenate([v[:-1][free], v[-1:]]) if op else v[:-1][free])
        got = np.concatenate([z[:-1][free], z[-1:]]) if op else z[free]
        assert relerr(got, ref) < (2e-4 if fp32 else tol)
        assert np.all((z[:-1] if op else z)[g.clamped_mask()] == 0)
        assert np.array_equal(z, N(s.vcycle(T(r), op=op)))


@pytest.mark.parametrize("nu", [(1, 0), (1, 1), (3, 2), (2, 3)])
@pytest.mark.parametrize("nel,levels,tail", [((40, 24), 4, True), ((40, 24), 4, False), ((12, 8, 4), 3, True),
                                             ((12, 8, 4), 3, False)])
def test_sweep_counts(nel, levels, tail, nu, monkeypatch):
    # other numbers of sweeps than 2 + 2: which of the two iterate buffers holds the
    # result, and the lambda entry's chain, depend on them
    from paper_1606_06201_amd import Solver
    prob = _problem(nel)
    g = prob.grid
    st, u_slots = _state(prob)
    Z, _, _ = prob.z_system(st)
    free = g.free_to_slot()
    if not tail:
        monkeypatch.setenv("IPMG_NO_TAIL", "1")
    s = Solver(nel, levels, fp32=False, nu_pre=nu[0], nu_post=nu[1])
    s.ip_prepare(T(prob.f_slots), s.ip_params(prob.V, prob.xbar), _gpu_state(s, st, u_slots))
    s.mg_setup(1)
    v = np.random.default_rng(4).standard_normal(g.nslots + 1)
    v[:-1][g.clamped_mask()] = 0
    z = N(s.vcycle(T(v), op=1))
    ref = mg.vcycle(mg.Hierarchy(g, Z, levels, augmented=True), np.concatenate([v[:-1][free], v[-1:]]), *nu)
    assert relerr(np.concatenate([z[:-1][free], z[-1:]]), ref) < 1e-9


@pytest.mark.parametrize("nel,levels", [((8, 4), 2), ((64, 32), 4), ((64, 32), 2), ((8, 4, 4), 3)])
@pytest.mark.parametrize("fp32", [False, True])
def test_pcg_steps_ended_in_the_tail(nel, levels, fp32, monkeypatch):
    # The PCG step's update, stop test and ratio inside the one-workgroup V-cycle against
    # the separate kernels: counts within one (the sums are grouped differently), solutions
    # to the tolerance of the solve; zero steps, a step limit and a breakdown-free restart.
    from paper_1606_06201_amd import Solver
    g, K0 = grid_and_k0(nel)
    x = np.random.default_rng(5).uniform(1e-2, 1.0, g.m)
    f = T(fem.load_vector(g, tip_load(nel)))
    out = []
    for off in ("0", "1"):
        monkeypatch.setenv("IPMG_NO_TAIL", off)
        s = Solver(nel, levels, fp32=fp32)
        s.set_density(T(x))
        u, info = s.pcg(f, rtol=1e-10)
        assert info["true_relres"] <= 1e-10
        _, i0 = s.pcg(f, u0=u, rtol=1e-8)
        u3, i3 = s.pcg(f, rtol=1e-14, maxit=3, check=False)
        un, inf_n = s.pcg_noalloc(f, rtol=1e-10)
        assert i0["iters"] == 0 and i3["iters"] == 3 and np.array_equal(N(un), N(u))
        out.append((N(u), info["iters"], N(u3)))
    assert abs(out[0][1] - out[1][1]) <= 1
    assert relerr(out[0][0], out[1][0]) < 1e-8
    assert relerr(out[0][2], out[1][2]) < (1e-5 if fp32 else 1e-11)
    ref = opcg.mg_pcg(mg.kstiffness_hierarchy(g, x, K0, levels), fem.to_free(g, N(f)), rtol=1e-10)
    assert abs(out[0][1] - ref.iters) <= (2 if fp32 else 1)
