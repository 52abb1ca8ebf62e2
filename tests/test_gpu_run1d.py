"""Small 1D problems, whose steps are taken many to a launch by one workgroup
each: the smallest meshes, meshes of whole waves (52 cells) and one cell fewer
or more, and the largest (416 cells, eight waves).  Steps asked for together,
one by one, to the end time, by the allocation-free step and in a handle whose
larger problem sends all of them through the one-step kernel must give the same
bits, and the oracle's step."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import oproblem, natural_scales, scaled_err
from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [4, 5, 51, 52, 53, 104, 105, 415, 416]


def _problem(flux, nx, bc, t_end):
    spec = W.Spec(dim=1, flux=flux, nx=nx, bc_x=bc, t_end=t_end)
    r = np.random.default_rng(nx)
    a, phi = r.uniform(0.1, 0.3), r.uniform(0, 6)

    def u0(x, c):
        s = 0.6 + a * np.sin(2 * np.pi * x + phi)
        if flux != W.EULER:
            return s[None]
        return W.conserved_1d(s, 0.3 * np.cos(2 * np.pi * x), 0.7 + 0.1 * np.sin(2 * np.pi * x))
    return spec, W.project_1d(spec, u0)


CASES = [(W.ADVECTION, 0, W.PERIODIC), (W.BURGERS, 0, W.TRANSMISSIVE), (W.EULER, 0, W.REFLECTIVE),
         (W.EULER, 1, W.PERIODIC), (W.EULER, 1, W.TRANSMISSIVE), (W.EULER, 1, W.REFLECTIVE)]


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64, hw.F32_KAHAN, hw.F32])
@pytest.mark.parametrize("flux,charwise,bc", CASES)
def test_small_problems_every_way(flux, charwise, bc, prec):
    cfg = hw.default_config(1, precision=prec, characteristic=charwise)
    probs = [_problem(flux, nx, bc, 10.0) for nx in SIZES]
    n = len(probs)

    def run(specs, take):
        with hw.Handle([s for s, _ in specs], cfg) as h:
            for i, (_, st) in enumerate(specs):
                h.set_state(i, st)
            take(h)
            return [h.get_state(i) for i in range(n)]

    def same(a, b):
        for (x, tx), (y, ty) in zip(a, b):
            np.testing.assert_array_equal(x, y)
            assert tx == ty

    five = run(probs, lambda h: h.steps(5))
    same(run(probs, lambda h: [h.step() for _ in range(5)]), five)
    same(run(probs + [_problem(flux, 417, bc, 10.0)], lambda h: h.steps(5)), five)

    two = run(probs, lambda h: h.steps(2))
    # bars of the one-step kernel's wave edges: 1e-12 in FP64, 2e-5 in single
    # precision for two steps
    bar = 1e-12 if prec == hw.F64 else 2e-5
    for (spec, st), (got, t) in zip(probs, two):
        p, ref, tr = oproblem(spec, cfg), st, 0.0
        for _ in range(2):
            ax, ay = O.alpha(p, ref)
            dt = O.dt(p, ax, ay, cfg.cfl)
            ref, tr = O.step(p, ref, ax, ay, dt), tr + dt
        assert scaled_err(got, ref, natural_scales(spec, st)) < bar, (spec.nx, bc)
        assert abs(t - tr) <= bar * tr

    # to the end time (some five steps away for each), in one launch or many
    ends = [_problem(flux, nx, bc, t) for nx, (_, t) in zip(SIZES, five)]
    same(run(ends, lambda h: h.run_to_time()), run(ends, lambda h: [h.step() for _ in range(7)]))

    # the allocation-free step
    for (spec, st), (want, t) in zip(probs, run(probs, lambda h: h.steps(1))):
        x = torch.from_numpy(np.ascontiguousarray(st)).cuda()
        y, aux = torch.empty_like(x), torch.zeros(2, dtype=torch.float64, device="cuda")
        hw.step_noalloc(spec, cfg, x, y, dt_out=aux.data_ptr(), bad_out=aux.data_ptr() + 8, stream=None)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(y.cpu().numpy(), want)
        assert float(aux[0]) == t
