"""The 1D step kernel with two cells per lane, which handles of many waves take:
its waves write 116 cells, so meshes of one cell fewer, exactly and one more,
the smallest ones, and meshes whose last wave holds less than its halo, for
every law, reconstruction, boundary and precision.  Problems beside fillers
that bring the handle to two cells per lane must give the bits of the same
problems with one cell per lane, and the oracle's steps."""
import functools

import numpy as np
import pytest

import oracle as O
from gpu_util import oproblem, natural_scales, scaled_err
from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu

# 731 cells are more than one workgroup takes whole: without fillers the batch
# goes through the same kernel with one cell per lane
SIZES = [4, 5, 115, 116, 117, 121, 122, 127, 128, 231, 232, 233, 731]
FILL = 3001


def _problem(flux, nx, bc):
    spec = W.Spec(dim=1, flux=flux, nx=nx, bc_x=bc, t_end=10.0)
    r = np.random.default_rng(nx)
    a, k, phi = r.uniform(0.1, 0.3), r.integers(1, 3), r.uniform(0, 6)

    def u0(x, c):
        s = 0.6 + a * np.sin(2 * np.pi * k * x + phi) + 0.2 * (x > 0.4)
        if flux != W.EULER:
            return s[None]
        return W.conserved_1d(s, 0.3 * np.cos(2 * np.pi * x), 0.7 + 0.1 * np.sin(2 * np.pi * x))
    return spec, W.project_1d(spec, u0)


@functools.lru_cache(maxsize=None)
def _fillers():
    """How many problems of FILL cells bring SIZES to two cells per lane.  A
    workspace holds the list of a step's waves: each filler adds the same bytes
    (to within the alignment of some ten regions) but for the one with which the
    waves grow from 52 to 116 cells, when the list of some thousands shrinks to
    half."""
    cfg = hw.default_config(1)
    specs = [W.Spec(dim=1, flux=W.BURGERS, nx=nx, t_end=10.0) for nx in SIZES]
    fill = W.Spec(dim=1, flux=W.BURGERS, nx=FILL, t_end=10.0)
    size = [hw.Handle.workspace_bytes(specs + [fill] * n, cfg) for n in range(202)]
    grow = np.diff(size)
    usual = int(np.median(grow))
    short = np.flatnonzero(grow < usual - 6000)
    assert len(short) == 1, "the handle never comes to two cells per lane"
    return int(short[0]) + 1


CASES = [(W.ADVECTION, 0, W.PERIODIC), (W.BURGERS, 0, W.PERIODIC), (W.BURGERS, 0, W.TRANSMISSIVE)] + [
    (W.EULER, ch, bc) for ch in (0, 1) for bc in (W.PERIODIC, W.TRANSMISSIVE, W.REFLECTIVE)]


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64, hw.F32_KAHAN, hw.F32])
@pytest.mark.parametrize("flux,charwise,bc", CASES)
def test_wave_edges_with_two_cells_per_lane(flux, charwise, bc, prec):
    cfg = hw.default_config(1, precision=prec, characteristic=charwise)
    probs = [_problem(flux, nx, bc) for nx in SIZES]
    fill = [_problem(flux, FILL, bc)] * _fillers()
    outs = []
    for specs, grid in ((probs, 0), (probs + fill, 0), (probs + fill, 301)):
        with hw.Handle([s for s, _ in specs], cfg) as h:
            h.set_tuning(grid_blocks=grid)
            for i, (_, st) in enumerate(specs):
                h.set_state(i, st)
            dts = h.step(want_dt=True)[:len(probs)]
            h.steps(1)
            outs.append(([h.get_state(i) for i in range(len(probs))], dts))
    for got, dts in outs[1:]:
        np.testing.assert_array_equal(dts, outs[0][1])
        for (spec, _), (a, ta), (b, tb) in zip(probs, got, outs[0][0]):
            np.testing.assert_array_equal(a, b, err_msg=f"{spec.nx} cells")
            assert ta == tb
    # two steps: 1e-12 in FP64; single precision rounds every stage with 6e-8
    # times the 30x cancellation of the reconstruction, and the derivative planes
    # add ~100 roundings of the flux terms (2e-5)
    bar = 1e-12 if prec == hw.F64 else 2e-5
    for (spec, st), (got, t) in zip(probs, outs[1][0]):
        p, ref, tr = oproblem(spec, cfg), st, 0.0
        for _ in range(2):
            ax, ay = O.alpha(p, ref)
            dt = O.dt(p, ax, ay, cfg.cfl)
            ref, tr = O.step(p, ref, ax, ay, dt), tr + dt
        assert scaled_err(got, ref, natural_scales(spec, st)) < bar, spec.nx
        assert abs(t - tr) <= bar * tr
