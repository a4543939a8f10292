"""Path switches act on their value: a switch at 0, or a size at its default, leaves the
default path, bit for bit; and the paths that a switch chooses on all levels are reached
with the one-workgroup V-cycle of small levels off."""
import numpy as np
import pytest

from tests.gpu_util import T, N, relerr, grid_and_k0

pytestmark = pytest.mark.gpu

OFF = [("IPMG_STORED_COARSE", "0"), ("IPMG_UNTILED", "0"), ("IPMG_UNFUSED", "0"), ("IPMG_UNSTAGED", "0"),
       ("IPMG_NO_MFMA", "0"), ("IPMG_NO_FOLD_RESTRICT", "0"), ("IPMG_NO_ELEM_FINE3", "0"), ("IPMG_NO_ELEM_HV", "0"),
       ("IPMG_NO_TAIL", "0"), ("IPMG_TILED_MIN_NODES", str(1 << 17)), ("IPMG_STAGED_MAX_NODES", str(1 << 16))]


def _vcycle(nel, levels, fp32, seed=5):
    from paper_1606_06201_amd import Solver
    g, _ = grid_and_k0(nel)
    rng = np.random.default_rng(seed)
    s = Solver(nel, levels, fp32=fp32)
    s.set_density(T(rng.uniform(0.01, 1.0, g.m)))
    s.mg_setup()
    return N(s.vcycle(T(rng.standard_normal(g.nslots))))


@pytest.mark.parametrize("nel,levels,fp32", [((64, 32), 4, True), ((160, 80), 4, False), ((12, 8, 4), 3, True)])
def test_switch_off_is_the_default(nel, levels, fp32, monkeypatch):
    ref = _vcycle(nel, levels, fp32)
    for env, val in OFF:
        monkeypatch.setenv(env, val)
        assert np.array_equal(_vcycle(nel, levels, fp32), ref), env
        monkeypatch.delenv(env)


@pytest.mark.parametrize("nel,levels", [((256, 128), 4), ((96, 48), 3), ((72, 40), 3)])
def test_first_coarse_level_matrix_cores(nel, levels, monkeypatch):
    # element products on the matrix cores against the vector units on ragged tiles: chained
    # FMAs in the same order, so equal to FP32 rounding
    monkeypatch.setenv("IPMG_NO_TAIL", "1")
    z = _vcycle(nel, levels, True)
    monkeypatch.setenv("IPMG_NO_MFMA", "1")
    assert relerr(z, _vcycle(nel, levels, True)) < 1e-6
