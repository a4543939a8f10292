"""3D grids at the largest number of node blocks whose partial sums have a slot each
(65536): one just below it is taken, one just above it is refused by every call whose
kernels leave a partial per node block, before any of them is launched."""
import numpy as np
import pytest

from oracle import fem
from tests.gpu_util import T, N, relerr

pytestmark = pytest.mark.gpu


def _blocks(nel):
    return -(-(nel[0] + 1) // 64) * -(-(nel[1] + 1) // 4) * (nel[2] + 1)


def _state(s):
    one = T(np.ones(s.m))
    return dict(u=T(np.random.default_rng(2).standard_normal(s.n_slots)), x=0.5 * one, phi=one.clone(),
                psi=one.clone(), lam=0.7, s=0.3, r=0.2)


def test_below_the_limit_is_taken():
    from paper_1606_06201_amd import Solver
    nel = (2, 512, 506)
    assert _blocks(nel) <= 65536
    s = Solver(nel, 2, fp32=True)
    g = fem.Grid(nel)
    st = _state(s)
    rhs = s.ip_prepare(st["u"], s.ip_params(0.5 * s.m), st)
    assert np.all(np.isfinite(N(rhs)))
    y = N(s.apply_K(st["u"]))
    assert relerr(y, fem.apply_free_masked(g, np.full(g.m, 0.5), fem.element_stiffness(3), N(st["u"]))) < 1e-13


def test_above_the_limit_is_refused():
    from paper_1606_06201_amd import Solver, _lib as L
    from paper_1606_06201_amd.solver import IPMGError
    nel = (2, 512, 512)
    assert _blocks(nel) > 65536
    s = Solver(nel, 2, fp32=True)
    st = _state(s)
    s.set_density(st["x"])
    f = T(np.zeros(s.n_slots))
    p = s.ip_params(0.5 * s.m)
    for call in (lambda: s.apply_K(st["u"]), lambda: s.ip_prepare(f, p, st), lambda: s.ip_step(f, p, st),
                 lambda: s.ip_step(f, p, st, simp=(2.0, 3.0)), lambda: s.pcg(st["u"])):
        with pytest.raises(IPMGError) as e:
            call()
        assert e.value.code == L.E_INVALID
