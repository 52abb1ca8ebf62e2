"""The one-kernel 1D step at the edges of its waves: a wave writes 52, 116 or
244 cells (1, 2 or 4 per lane, by the total size), so meshes of one cell
fewer, exactly, and one cell more, the smallest mesh, and meshes whose last
wave holds less than its halo, under every boundary.  The oracle's step is
the reference; problems of a batch and a persistent grid must give the bits
of a problem alone."""
import numpy as np
import pytest

import oracle as O
from gpu_util import oproblem, natural_scales, scaled_err
from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [4, 5, 51, 52, 53, 57, 105, 116, 117, 122, 244, 245, 731]


def _problem(nx, bc, seed):
    spec = W.Spec(dim=1, flux=W.EULER, nx=nx, bc_x=bc, t_end=10.0)
    r = np.random.default_rng(seed)
    a, k, phi = r.uniform(0.1, 0.3), r.integers(1, 3), r.uniform(0, 6)

    def u0(x, c):
        rho = 0.6 + a * np.sin(2 * np.pi * k * x + phi) + 0.2 * (x > 0.4)
        return W.conserved_1d(rho, 0.3 * np.cos(2 * np.pi * x), 0.7 + 0.1 * np.sin(2 * np.pi * x))
    return spec, W.project_1d(spec, u0)


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64, hw.F32_KAHAN, hw.F32])
@pytest.mark.parametrize("charwise", [0, 1])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.TRANSMISSIVE, W.REFLECTIVE])
def test_wave_edges(bc, charwise, prec):
    cfg = hw.default_config(1, precision=prec, characteristic=charwise)
    probs = [_problem(nx, bc, nx) for nx in SIZES]
    # fillers bring the batch to two cells per lane
    fill = [_problem(3001, bc, 1)] * 40
    outs = []
    for specs, grid in ((probs, 0), (probs, 7), (probs + fill, 0)):
        with hw.Handle([s for s, _ in specs], cfg) as h:
            h.set_tuning(grid_blocks=grid)
            for i, (_, st) in enumerate(specs):
                h.set_state(i, st)
            dts = h.step(want_dt=True)[:len(probs)]
            h.steps(1)
            outs.append(([h.get_state(i) for i in range(len(probs))], dts))
    for got, dts in outs[1:]:
        np.testing.assert_array_equal(dts, outs[0][1])
        for (a, ta), (b, tb) in zip(got, outs[0][0]):
            np.testing.assert_array_equal(a, b)
            assert ta == tb
    # bars of one operator step: 1e-12 in FP64; single precision rounds every
    # stage with 6e-8 times the 30x cancellation of the reconstruction, and the
    # derivative planes add ~100 roundings of the flux terms (2 steps: 2e-5)
    bar = 1e-12 if prec == hw.F64 else 2e-5
    for (spec, st), (got, t) in zip(probs, outs[0][0]):
        p, ref, tr = oproblem(spec, cfg), st, 0.0
        for _ in range(2):
            ax, ay = O.alpha(p, ref)
            dt = O.dt(p, ax, ay, cfg.cfl)
            ref, tr = O.step(p, ref, ax, ay, dt), tr + dt
        assert scaled_err(got, ref, natural_scales(spec, st)) < bar, (spec.nx, bc)
        assert abs(t - tr) <= bar * tr
