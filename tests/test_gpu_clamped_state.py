"""Entries of a displacement state at clamped nodes are ignored by every call that takes
one: the Newton system and a Newton step come out the same, bit for bit, whatever stands
there."""
import numpy as np
import pytest

from oracle import fem
from tests.gpu_util import T, N
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu

VALUES = (0.0, 7.5, np.nan)


def _with_clamped(g, u, value):
    u = u.copy()
    u[g.clamped_mask()] = value
    return u


@pytest.mark.parametrize("nel", [(12, 8), (12, 8, 4), (34, 10, 4)])
@pytest.mark.parametrize("fp32", [False, True])
def test_newton_system(nel, fp32):
    from paper_1606_06201_amd import Solver
    prob = _problem(nel)
    g = prob.grid
    st, u = _state(prob)
    v = T(np.random.default_rng(3).standard_normal(g.nslots + 1))
    out = []
    for value in VALUES:
        s = Solver(nel, 2, fp32=fp32)
        rhs = s.ip_prepare(T(prob.f_slots), s.ip_params(prob.V, prob.xbar),
                           _gpu_state(s, st, _with_clamped(g, u, value)))
        out.append(np.concatenate([N(rhs), N(s.apply_Z(v))]))
    assert all(np.array_equal(o, out[0]) for o in out)


@pytest.mark.parametrize("nel", [(12, 8), (12, 8, 4)])
@pytest.mark.parametrize("simp", [None, (2.0, 3.0)])
def test_newton_step(nel, simp):
    from paper_1606_06201_amd import Solver
    prob = _problem(nel, vfrac=0.4, xbar=3.0)
    g = prob.grid
    f = T(prob.f_slots)
    out = []
    for value in VALUES:
        s = Solver(nel, 2, fp32=False)
        p = s.ip_params_paper(prob.V, xbar=3.0)
        st, _ = s.ip_init(f, p, simp=simp)
        st["u"] = T(_with_clamped(g, N(st["u"]), value))
        inf = s.ip_step(f, p, st, simp=simp)
        assert inf["rc"] == 0
        out.append(np.concatenate([N(st["x"]), N(st["phi"]), N(st["psi"]), fem.to_free(g, N(st["u"])),
                                   [st["lam"], inf["alpha"], inf["nwt"], inf["gap"], inf["compliance"]]]))
    assert all(np.array_equal(o, out[0]) for o in out)
