"""What ipmg_pcg reports of a solve that did not converge: its relres is never within the
tolerance, since a stop of the recurrence is confirmed with the true residual and a restart
goes on from that one."""
import numpy as np
import pytest

from oracle import fem
from tests.gpu_util import T, tip_load

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,levels,seed", [((64, 32), 4, 6), ((64, 32), 2, 5), ((160, 80), 4, 5)])
def test_relres_of_a_breakdown(nel, levels, seed):
    # Loads near 1e-30: the residual that a restart begins with is at the smallest floats,
    # so that the FP32 V-cycle of it can be no descent direction (r'y <= 0) at once.
    from paper_1606_06201_amd import Solver, _lib as L
    g = fem.Grid(nel)
    s = Solver(nel, levels, fp32=True)
    s.set_density(T(np.random.default_rng(seed).uniform(0.01, 1.0, g.m)))
    f = T(fem.load_vector(g, tip_load(nel)))
    stopped = 0
    for e in np.arange(-32.0, -28.0, 0.25):
        for rtol in 10.0 ** np.arange(-14.0, -11.0, 0.5):
            _, i = s.pcg(10.0**e * f, rtol=float(rtol), maxit=60, check=False)
            if i["rc"] == L.OK:
                assert i["true_relres"] <= rtol
            else:
                stopped += i["rc"] == L.E_BREAKDOWN
                assert i["relres"] > rtol, (e, rtol, i)
    assert stopped > 0
