"""The density filter with its column sums looked up by the distance to the edges:
grids no wider than the neighbourhood, one element wider, the widest neighbourhood, and
Newton steps on grids whose whole V-cycle is one workgroup's and on larger ones."""
import numpy as np
import pytest

from oracle import fem, simp
from tests.gpu_util import T, N, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,rmin", [((2, 2), 5.0), ((8, 2), 5.0), ((9, 10), 5.0), ((10, 9), 4.5), ((33, 17), 1.5),
                                      ((2, 4, 2), 3.0), ((9, 8, 10), 5.0), ((12, 5, 3), 4.0), ((4, 4, 4), 0.5)])
def test_filter_at_the_edges(nel, rmin):
    from paper_1606_06201_amd import Solver
    g = fem.Grid(nel)
    W = simp.filter_matrix(g, rmin)
    v = np.random.default_rng(7).uniform(0.1, 1.0, g.m)
    s = Solver(nel, 1, fp32=False)
    # positive terms: a row sum, its column sums and their quotient, to eps a term
    terms = 2 * int(np.ceil(rmin)) + 1
    tol = 3 * terms ** len(nel) * np.finfo(float).eps
    assert relerr(N(s.filter(T(v), rmin)), W @ v) < tol
    assert relerr(N(s.filter(T(v), rmin, transpose=True)), W.T @ v) < tol


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("nel,levels", [((16, 8), 3), ((16, 8), 1), ((64, 32), 5), ((8, 4, 4), 2)])
def test_simp_newton_steps_match_oracle(nel, levels, fp32):
    # systems solved to 1e-11, the oracle's directly: the tolerances of the step test at
    # one grid, for both precisions and the forms of the V-cycle
    from oracle import ip as oip
    from paper_1606_06201_amd import Solver, inputs
    g = fem.Grid(nel)
    f = fem.load_vector(g, inputs.point_load(nel))
    prob = simp.SimpProblem(g, fem.element_stiffness(g.dim), f, 0.4 * g.m, 3.0, rmin=2.0, p=3.0)
    po = oip.IPParams(solver="direct")
    st_o, _ = oip.initial_state(prob, po)
    s = Solver(nel, levels, fp32=fp32)
    params = s.ip_params(prob.V, prob.xbar, pcg_rtol=1e-11, pcg_maxit=4000)
    st, _ = s.ip_init(T(prob.f_slots), params, simp=(2.0, 3.0))
    for k in range(2):
        inf = s.ip_step(T(prob.f_slots), params, st, simp=(2.0, 3.0))
        st_o, alpha_o, _ = oip.newton_step(prob, st_o, po)
        print(nel, levels, fp32, k, inf["pcg_iters"], inf["alpha"], alpha_o, flush=True)
        assert inf["rc"] == 0 and inf["pcg_status"] == 0
        assert abs(inf["alpha"] - alpha_o) <= 1e-7
        assert relerr(N(st["x"]), st_o.x) < 1e-7
        assert relerr(fem.to_free(g, N(st["u"])), st_o.u) < 1e-7
