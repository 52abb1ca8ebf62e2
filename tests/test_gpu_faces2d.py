"""The 2D stage kernels at the edges of their strips (60 columns) and segments,
for every law, number of Gauss points and precision: a scalar law keeps its
faces in registers, Euler passes them through LDS, and the characteristic
kernel projects them; the rows beside a segment lend it one edge only.  Meshes
down to four cells under every pair of boundaries; the reference is the
oracle's step."""
import numpy as np
import pytest

import oracle as O
from gpu_util import oproblem, natural_scales, scaled_err
from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu

MESHES = [(4, 4, W.PERIODIC, W.TRANSMISSIVE), (59, 5, W.TRANSMISSIVE, W.PERIODIC),
          (60, 6, W.PERIODIC, W.PERIODIC), (61, 7, W.TRANSMISSIVE, W.TRANSMISSIVE),
          (121, 33, W.PERIODIC, W.TRANSMISSIVE)]
WALLS = [(5, 4, W.REFLECTIVE, W.PERIODIC), (62, 9, W.REFLECTIVE, W.REFLECTIVE)]


def _problem(flux, nx, ny, bcx, bcy):
    spec = W.Spec(dim=2, flux=flux, nx=nx, ny=ny, bc_x=bcx, bc_y=bcy, t_end=10.0)

    def u0(x, y, i, j):
        s = 0.7 + 0.2 * np.sin(2 * np.pi * (x + y) + 0.4)
        if flux != W.EULER:
            return s[None]
        u, v = 0.3 * np.cos(2 * np.pi * x), -0.2 * np.sin(2 * np.pi * y)
        p = 0.8 + 0.1 * np.cos(2 * np.pi * (x - y))
        return np.stack([s, s * u, s * v, p / 0.4 + 0.5 * s * (u * u + v * v)])
    return spec, W.project_2d(spec, u0)


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64, hw.F32_KAHAN, hw.F32])
@pytest.mark.parametrize("q", [2, 3])
@pytest.mark.parametrize("flux,charwise", [(W.ADVECTION, 0), (W.BURGERS, 0), (W.EULER, 0), (W.EULER, 1)])
def test_strip_and_segment_edges(flux, charwise, q, prec):
    cfg = hw.default_config(2, precision=prec, gauss_q=q, characteristic=charwise)
    # one step: 1e-12 in FP64, in single precision the bar of the 2D step there
    bar = 1e-12 if prec == hw.F64 else 4e-4
    for mesh in MESHES + (WALLS if flux == W.EULER else []):
        spec, st = _problem(flux, *mesh)
        with hw.Handle([spec], cfg) as h:
            h.set_state(0, st)
            dt = h.step(want_dt=True)[0]
            got, t = h.get_state(0)
            ax, ay = h.alpha(0)
        p = oproblem(spec, cfg)
        rx, ry = O.alpha(p, st)
        assert dt == O.dt(p, rx, ry, cfg.cfl) == t or prec != hw.F64
        assert scaled_err(got, O.step(p, st, rx, ry, dt), natural_scales(spec, st)) < bar, mesh
        # the speeds gathered from the new state are those of its averages
        assert (ax, ay) == tuple(O.alpha(p, got)), mesh
