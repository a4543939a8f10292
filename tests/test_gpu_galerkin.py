"""Galerkin products and the dense coarsest operator at the sizes where their kernels
change: 64 coarse elements of the first coarse level in 3D, 1024 of the next ones, and
coarsest orders of one tile and several.  The spectral radii of the levels and a V-cycle
follow the oracle's to 1e-9: FP64 rounding times the condition number of the coarsest
operator, as for the V-cycle of the augmented system elsewhere."""
import numpy as np
import pytest

from oracle import mg
from tests.gpu_util import T, N, relerr, grid_and_k0
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,levels", [((128, 128), 3), ((136, 128), 3), ((24, 8), 3), ((16, 16, 16), 3),
                                        ((12, 8, 8), 2), ((8, 8, 8), 2), ((24, 16, 8), 4), ((20, 12, 8), 3)])
def test_coarse_operators(nel, levels):
    from paper_1606_06201_amd import Solver
    prob = _problem(nel)
    g = prob.grid
    st, u_slots = _state(prob)
    Z, _, _ = prob.z_system(st)
    _, K0 = grid_and_k0(nel)
    free = g.free_to_slot()
    s = Solver(nel, levels, fp32=False)
    s.ip_prepare(T(prob.f_slots), s.ip_params(prob.V, prob.xbar), _gpu_state(s, st, u_slots))
    v = np.random.default_rng(8).standard_normal(g.nslots + 1)
    v[:-1][g.clamped_mask()] = 0
    for op, H in ((1, mg.Hierarchy(g, Z, levels, augmented=True)), (0, mg.kstiffness_hierarchy(g, st.x, K0, levels))):
        s.mg_setup(op)
        for k in range(1, levels):
            assert abs(s.level_damping(k)[1] - H.rho[k]) <= 1e-9 * H.rho[k]
        z = N(s.vcycle(T(v if op else v[:-1]), op=op))
        ref = mg.vcycle(H, np.concatenate([v[:-1][free], v[-1:]]) if op else v[:-1][free])
        assert relerr(np.concatenate([z[:-1][free], z[-1:]]) if op else z[free], ref) < 1e-9
