"""Solvers of different materials in one process: each gives what it gives alone, bit for
bit, whichever was made last, called in turn and from two threads at once."""
import threading

import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, T, N
from tests.test_gpu_ip import _gpu_state, _problem, _state

pytestmark = pytest.mark.gpu

MATERIALS = [dict(E=1.0, nu=0.3), dict(E=2.5, nu=0.1)]
NAMES = ["rhs", "Z v", "K v", "sens", "V-cycle Z", "V-cycle K", "u", "oc"]


def _calls(s, prob, st, u, v):
    f = T(prob.f_slots)
    out = [s.ip_prepare(f, s.ip_params(prob.V, prob.xbar), _gpu_state(s, st, u)), s.apply_Z(T(v)), s.apply_K(T(v[:-1])),
           s.element_sens(T(v[:-1]), T(u))]
    s.mg_setup(1)
    out.append(s.vcycle(T(v), op=1))
    s.mg_setup(0)
    out += [s.vcycle(T(v[:-1]), op=0), s.pcg(f, rtol=1e-10)[0]]
    out.append(s.oc_update(T(u), T(st.x), prob.V, 1.0)[0])
    return [N(o) for o in out]


@pytest.mark.parametrize("nel,levels", [((16, 8), 3), ((160, 80), 5), ((16, 8, 8), 3)])
@pytest.mark.parametrize("fp32", [False, True])
def test_in_turn(nel, levels, fp32):
    from paper_1606_06201_amd import Solver
    prob = _problem(nel)
    st, u = _state(prob)
    v = np.random.default_rng(3).standard_normal(prob.grid.nslots + 1)
    v[:-1][prob.grid.clamped_mask()] = 0
    ref = []
    for mat in MATERIALS:
        s = Solver(nel, levels, fp32=fp32, **mat)
        ref.append(_calls(s, prob, st, u, v))
        s.close()
    assert not np.array_equal(ref[0][2], ref[1][2])
    both = [Solver(nel, levels, fp32=fp32, **mat) for mat in MATERIALS]
    for k in (0, 1, 1, 0):
        got = _calls(both[k], prob, st, u, v)
        assert [n for n, a, b in zip(NAMES, got, ref[k]) if not np.array_equal(a, b)] == []


def test_from_two_threads():
    from paper_1606_06201_amd import Solver
    nel, levels = (16, 8, 8), 3
    prob = _problem(nel)
    x, f = T(np.random.default_rng(5).uniform(0.1, 1.0, prob.grid.m)), T(prob.f_slots)
    torch.cuda.synchronize()

    def solver(mat):
        st = torch.cuda.Stream(DEV)
        with torch.cuda.stream(st):
            return Solver(nel, levels, fp32=True, **mat), st

    def solve(pair):
        s, st = pair
        with torch.cuda.stream(st):
            s.set_density(x)
            return N(s.pcg(f, rtol=1e-10)[0])

    ss = [solver(mat) for mat in MATERIALS + MATERIALS[:1]]      # two of the first material
    ref = [solve(s) for s in ss]
    bad = []

    def work(k):
        for _ in range(15):
            if not np.array_equal(solve(ss[k]), ref[k]):
                bad.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(ss))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
    assert not any(t.is_alive() for t in ts) and bad == []
