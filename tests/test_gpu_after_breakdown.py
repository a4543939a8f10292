"""A solve after one that broke down, on the same solver: nothing of the failed one is left
in it, so the result is the first one's, bit for bit.  Loads from just below to far above
what the V-cycle's precision and the squares of FP64 hold."""
import numpy as np
import pytest

from oracle import fem
from tests.gpu_util import T, N, tip_load, grid_and_k0

pytestmark = pytest.mark.gpu

SCALES = [1e30, 3e36, 1e37, 1e38, 1e39, 1e148, 1e150, 1e152, 1e153, 3e153, 1e154, 1e200]


@pytest.mark.parametrize("nel,levels", [((64, 32), 4), ((160, 80), 4), ((512, 272), 5), ((16, 8, 8), 3), ((34, 10, 10), 2)])
@pytest.mark.parametrize("fp32", [False, True])
def test_solve(nel, levels, fp32):
    from paper_1606_06201_amd import Solver, _lib as L
    g, _ = grid_and_k0(nel)
    s = Solver(nel, levels, fp32=fp32)
    s.set_density(T(np.random.default_rng(5).uniform(0.01, 1.0, g.m)))
    f = T(fem.load_vector(g, tip_load(nel)))
    ref, broke = N(s.pcg(f, rtol=1e-8)[0]), 0
    for scale in SCALES:
        _, info = s.pcg(scale * f, rtol=1e-8, maxit=60, check=False)
        broke += info["rc"] == L.E_BREAKDOWN
        assert np.array_equal(N(s.pcg(f, rtol=1e-8)[0]), ref), scale
    assert broke > 0


@pytest.mark.parametrize("nel,levels", [((64, 32), 5), ((8, 4, 4), 2)])
@pytest.mark.parametrize("simp", [None, (2.0, 3.0)])
def test_newton_step(nel, levels, simp):
    from paper_1606_06201_amd import Solver, IPMGError
    g, _ = grid_and_k0(nel)
    f = T(fem.load_vector(g, tip_load(nel)))
    s = Solver(nel, levels, fp32=True)
    p = s.ip_params_paper(0.4 * g.m, xbar=3.0)

    def step(scale):
        st, _ = s.ip_init(f, p, simp=simp)
        inf = s.ip_step(scale * f, p, st, simp=simp)
        return inf["rc"], np.concatenate([N(st["x"]), N(st["u"])])

    rc, ref = step(1.0)
    assert rc == 0
    for scale in SCALES:
        try:
            step(scale)
        except IPMGError:
            pass
        rc, got = step(1.0)
        assert rc == 0 and np.array_equal(got, ref), scale
