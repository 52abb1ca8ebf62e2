"""Rounding of the 2D kernels where a coarse bar against the FP64 oracle, which
rounds as much itself, cannot see it."""
import numpy as np
import pytest

from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64])
def test_hats_of_linear_fields(prec):
    """On a linear field every candidate polynomial is the field itself, so the
    modified derivatives are its slopes whatever the weights.  With slopes of a
    few bits every sum and difference is exact, and what remains is the rounding
    of the product with the weights' sum: half a unit if that is 1, as it is for
    the default linear weights (in single precision the reciprocal may be off by
    a unit).  Weights that sum to one only to within two units would show in
    every cell."""
    n = 12
    slopes = [(k * 2.0 ** -8, (32 - k) * 2.0 ** -7) for k in range(1, 32, 2)]
    spec = W.Spec(dim=2, flux=W.ADVECTION, nx=n, ny=n, bc_x=W.TRANSMISSIVE, bc_y=W.TRANSMISSIVE,
                  t_end=1.0)
    bar = 2.0 ** -53 if prec == hw.F64 else 1.5 * 2.0 ** -23
    with hw.Handle([spec] * len(slopes), hw.default_config(2, precision=prec)) as h:
        for p, (sx, sy) in enumerate(slopes):
            st = np.empty((3, 1, n, n))
            st[0, 0] = sx * np.arange(n)[None, :] + sy * np.arange(n)[:, None]
            st[1], st[2] = sx, sy    # scaled averages: differences over a cell
            h.set_state(p, st)
        for p, s in enumerate(slopes):
            hats = h.rhs(p)[1]
            for v in (1, 2):
                err = np.abs(hats[v, 0, 1:-1, 1:-1] / s[v - 1] - 1.0).max()
                assert err <= bar, (s, v, err)
