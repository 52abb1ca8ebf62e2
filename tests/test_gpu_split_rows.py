"""Segment heights of small 2D problems: with one workgroup per tile the
library cuts a problem that would not fill the GPU into shorter segments than
tile_rows, of uneven heights where they do not divide the mesh.  A persistent
grid keeps the caller's heights, so the two must give the same bits, and the
oracle's step."""
import numpy as np
import pytest

import oracle as O
from gpu_util import oproblem, natural_scales, scaled_err
from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("charwise", [0, 1])
@pytest.mark.parametrize("nx,ny", [(4, 4), (61, 5), (60, 13), (121, 97), (64, 259)])
def test_short_segments_equal_the_callers_heights(nx, ny, charwise):
    entries = W.batched_2d(seed=nx + ny, nprob=1, nmin=max(nx, ny), nmax=max(nx, ny))
    spec, st = entries[0][0], W.batched_2d_state(entries[0])
    spec = W.replace(spec, nx=nx, ny=ny, bc_x=W.PERIODIC, bc_y=W.TRANSMISSIVE)
    st = np.ascontiguousarray(st[:, :, :ny, :nx])
    cfg = hw.default_config(2, precision=hw.F64, gauss_q=3, characteristic=charwise)
    outs = []
    for rows, grid in ((32, 0), (8, 0), (32, 5), (1024, 0)):
        with hw.Handle([spec], cfg) as h:
            h.set_tuning(tile_rows=rows, grid_blocks=grid)
            h.set_state(0, st)
            dt = h.step(want_dt=True)[0]
            outs.append((h.get_state(0)[0], dt))
    for o, d in outs[1:]:
        np.testing.assert_array_equal(o, outs[0][0])
        assert d == outs[0][1]
    p = oproblem(spec, cfg)
    ax, ay = O.alpha(p, st)
    # the bar of every FP64 step against the oracle
    assert scaled_err(outs[0][0], O.step(p, st, ax, ay, outs[0][1]), natural_scales(spec, st)) < 1e-12
