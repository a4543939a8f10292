"""The bisection of the OC update against the oracle's at the sizes where its kernels
change: elements per thread of the one-workgroup form, its last size, the passes past
it, and multipliers too small for the reciprocal form of the quotient."""
import numpy as np
import pytest

from oracle import fem, oc as ooc
from tests.gpu_util import T, N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,levels,scale,blend", [
    ((2, 2), 1, 1.0, False), ((64, 32), 5, 1.0, True), ((66, 32), 2, 1.0, False), ((128, 64), 6, 1.0, True),
    ((130, 64), 2, 1.0, False), ((128, 128), 6, 1.0, True), ((130, 128), 2, 1.0, False), ((256, 192), 6, 1.0, True),
    ((64, 32), 5, 1e-75, False), ((256, 192), 6, 1e-75, False), ((16, 8, 8), 3, 1.0, False)])
def test_bisection_matches_oracle(nel, levels, scale, blend):
    from paper_1606_06201_amd import Solver
    g = fem.Grid(nel)
    rng = np.random.default_rng(5)
    x = rng.uniform(0.05, 1.0, g.m)
    s = Solver(nel, levels, fp32=False)
    u_slots = fem.to_slots(g, fem.to_free(g, rng.standard_normal(s.n_slots)))
    ue = fem.element_values(g, u_slots)
    K0 = fem.element_stiffness(g.dim)
    E = np.einsum("ei,ij,ej->e", ue, K0, ue)
    V, xbar, hi, tau = x.sum(), 2.0, 1e4, 1e-11
    # the energies are computed to 64 eps ||K0|| ||u_e||^2, a sum of m terms to m eps of it
    d_e = 64 * np.finfo(float).eps * np.linalg.norm(K0, 2) * np.einsum("ei,ei->e", ue, ue) / E
    xo, lam, trials = ooc.bisect(x * E, V, xbar, hi, tau)
    free = xo < xbar
    d_lam = (np.sum((xo * d_e)[free]) + g.m * np.finfo(float).eps * V) / np.sum(xo[free]) + 2 * tau / lam
    u_gpu = scale * u_slots
    b = rng.uniform(0.05, 1.0, g.m) if blend else None
    xn, info = s.oc_update(T(u_gpu), T(x), V, xbar, 1.0, hi * scale ** 2, tau * scale ** 2,
                           blend=None if b is None else T(b))
    xg = N(xn)
    want = xo if b is None else 0.5 * (b + xo)
    print(nel, scale, info, lam, d_lam, float(np.max(np.abs(xg - want))), flush=True)
    assert info["trials"] == trials
    assert abs(info["lam"] - lam * scale ** 2) <= d_lam * lam * scale ** 2
    assert np.all(np.abs(xg - want) <= (d_e + d_lam + 1e-15) * want)
    assert abs(info["volume"] - xg.sum()) <= g.m * np.finfo(float).eps * V
