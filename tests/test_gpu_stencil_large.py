"""Augmented-system levels of more than 2048 stencil tiles, whose lambda entries are summed
by launches of their own and whose first sweep is separate, and a finest level above the
stencil sizes over stencil levels, against the FP64 oracle.  Bounds as for the smaller
grids: FP64 1e-9 or what rounding of the coarsest operator allows (eps times its condition
number, 7e9 on the slender grid), FP32 2e-4, damping estimates 1e-9 and 1e-4."""
import numpy as np
import pytest

from oracle import mg
from tests.gpu_util import T, N, relerr
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu

# 2049 tiles (one past the line) and 2189; 577 x 513 nodes, past 2^18, over levels below it
GRIDS = [((2016, 64), 6), ((512, 272), 5), ((576, 512), 6)]


@pytest.fixture(scope="module")
def systems():
    made = {}

    def system(nel, levels):
        if nel not in made:
            prob = _problem(nel)
            st, u_slots = _state(prob)
            Z, _, _ = prob.z_system(st)
            H = mg.Hierarchy(prob.grid, Z, levels, augmented=True)
            ev = np.linalg.eigvalsh(H.A[0].toarray())
            made[nel] = prob, st, u_slots, H, max(1e-9, np.finfo(float).eps * ev[-1] / ev[0])
        return made[nel]

    return system


@pytest.mark.parametrize("nel,levels", GRIDS)
@pytest.mark.parametrize("fp32,nu", [(True, (2, 2)), (False, (2, 2)), (False, (1, 1)), (False, (3, 2)), (False, (2, 0))])
def test_vcycle_and_solve(systems, nel, levels, fp32, nu):
    from paper_1606_06201_amd import Solver
    prob, st, u_slots, H, tol = systems(nel, levels)
    g = prob.grid
    free = g.free_to_slot()
    s = Solver(nel, levels, fp32=fp32, nu_pre=nu[0], nu_post=nu[1])
    s.ip_prepare(T(prob.f_slots), s.ip_params(prob.V, prob.xbar), _gpu_state(s, st, u_slots))
    s.mg_setup(1)
    for k in range(1, levels):
        assert abs(s.level_damping(k)[1] - H.rho[k]) <= (1e-4 if fp32 else 1e-9) * H.rho[k]
    v = np.random.default_rng(3).standard_normal(g.nslots + 1)
    v[:-1][g.clamped_mask()] = 0
    z = N(s.vcycle(T(v), op=1))
    ref = mg.vcycle(H, np.concatenate([v[:-1][free], v[-1:]]), *nu)
    assert relerr(np.concatenate([z[:-1][free], z[-1:]]), ref) < (2e-4 if fp32 else tol)
    assert np.all(z[:-1][g.clamped_mask()] == 0)
    if nu == (2, 2):
        # the PCG ratio formed in the last sweep, and its lambda entry, carry a solve
        u, info = s.pcg(T(v), op=1, rtol=1e-8, maxit=400)
        assert info["true_relres"] <= 1e-8
        r = N(s.apply_Z(u)) - v
        assert np.linalg.norm(r) <= 1.01e-8 * np.linalg.norm(v)
