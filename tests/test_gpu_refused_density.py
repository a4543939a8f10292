"""Densities that ip_prepare refuses leave the Newton system of the call before: with the
former densities set again, Z v and a solve on Z are what they were, bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import T, N
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,levels", [((12, 8), 2), ((12, 8, 4), 2), ((160, 80), 4)])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("value", [-1.0, 0.0, np.inf, np.nan])
def test_newton_system_is_kept(nel, levels, fp32, value):
    from paper_1606_06201_amd import Solver, _lib as L
    from paper_1606_06201_amd.solver import IPMGError
    prob = _problem(nel)
    st, u = _state(prob)
    f, v = T(prob.f_slots), T(np.random.default_rng(3).standard_normal(prob.grid.nslots + 1))
    s = Solver(nel, levels, fp32=fp32)
    p = s.ip_params(prob.V, prob.xbar)

    def outputs():
        s.mg_setup(1)
        return [N(s.apply_Z(v)), N(s.vcycle(v, op=1))]

    rhs = s.ip_prepare(f, p, _gpu_state(s, st, u))
    ref = outputs()
    bad = _gpu_state(s, st, 2.0 * u)
    bad["x"][prob.grid.m // 2] = value
    with pytest.raises(IPMGError) as e:
        s.ip_prepare(f, p, bad)
    assert e.value.code == L.E_DOMAIN and "densities" in str(e.value)
    with pytest.raises(IPMGError) as e:
        s.pcg(rhs, op=1)
    assert e.value.code == L.E_STATE
    s.set_density(T(st.x))
    assert all(np.array_equal(a, b) for a, b in zip(outputs(), ref))
    assert np.array_equal(N(s.ip_prepare(f, p, _gpu_state(s, st, u))), N(rhs))
