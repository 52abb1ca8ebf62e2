"""How many steps one launch of the many-step 1D kernel takes: a launch is not to
hold the GPU for long however many problems a handle has (the rule, called in the
library without a GPU), and steps that take several launches are the same steps."""
import numpy as np
import pytest

from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W


def _most(nprob):
    return hw.lib()._ZN5hweno11run1d_stepsEi(nprob)


def test_a_launch_is_bounded_whatever_the_number_of_problems():
    assert _most(1) == _most(256) == 4096
    for nprob in (257, 600, 1000, 4096, 100_000, 3_000_000):
        rounds = -(-nprob // 256)   # of workgroups, one to a CU
        assert 1 <= _most(nprob) and (_most(nprob) * rounds <= 4096 or _most(nprob) == 1)


@pytest.mark.gpu
def test_steps_across_launches():
    nprob = 600   # 1365 steps a launch
    most = _most(nprob)
    specs = [W.Spec(dim=1, flux=W.BURGERS, nx=4 + i % 5, t_end=1e9) for i in range(nprob)]
    x = [0.7 + 0.2 * np.sin(2 * np.pi * (np.arange(s.nx) + 0.5) / s.nx + i) for i, s in enumerate(specs)]
    outs = []
    for counts in ([most + 70], [most - 1, 71]):
        with hw.Handle(specs, hw.default_config(1)) as h:
            for i, u in enumerate(x):
                st = np.zeros((2, 1, 1, specs[i].nx))
                st[0, 0, 0] = u
                h.set_state(i, st)
            for n in counts:
                h.steps(n)
            outs.append([h.get_state(i) for i in range(nprob)])
    for (a, ta), (b, tb) in zip(*outs):
        np.testing.assert_array_equal(a, b)
        assert ta == tb > 0


@pytest.mark.gpu
def test_run_to_time_of_many_problems():
    nprob, t_end = 300, 0.5
    specs = [W.Spec(dim=1, flux=W.ADVECTION, nx=8 + i % 3, t_end=t_end * (1 + i % 4)) for i in range(nprob)]
    with hw.Handle(specs, hw.default_config(1)) as h:
        for i, s in enumerate(specs):
            st = np.ones((2, 1, 1, s.nx))
            st[1] = 0
            h.set_state(i, st)
        n = h.run_to_time()
        assert all(h.get_state(i)[1] == s.t_end for i, s in enumerate(specs))
    longest = max(s.t_end * s.nx for s in specs) / 0.6   # steps of 0.6 dx at speed one
    assert n == int(np.ceil(longest - 1e-9))
