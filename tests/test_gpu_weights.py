"""Every form of the nonlinear weights, and linear weights other than the
default, in every kernel that holds them: 1D problems stepped many to a launch,
one whole step per launch and stage by stage (the speeds of every stage), the
1D and 2D operators, and the 2D stage kernels component-wise and in
characteristic variables.  The oracle's operator and step are the reference."""
import numpy as np
import pytest

import oracle as O
from gpu_util import (oproblem, natural_scales, rhs_scales, oracle_sensitivity, scaled_err,
                      within_conditioning)
from paper_2607_24325_amd import hweno as hw
from paper_2607_24325_amd import workloads as W

pytestmark = pytest.mark.gpu

GAMMA = {1: (0.7, 0.1, 0.2, 0.0, 0.0), 2: (0.6, 0.1, 0.15, 0.05, 0.1)}
FORMS = [("paper", hw.W_PAPER, False), ("beta", hw.W_BETA, True), ("beta2", hw.W_BETA2, False),
         ("beta2-own", hw.W_BETA2, True), ("linear", hw.W_LINEAR, False)]


def _waves_1d(nx):
    """Waves of some twenty cells and a jump: barely resolved, so that the
    weights are far from the linear ones and each form gives its own"""
    spec = W.Spec(dim=1, flux=W.EULER, nx=nx, t_end=10.0)

    def u0(x, c):
        rho = 0.6 + 0.2 * np.sin(2 * np.pi * nx / 25 * x + 0.3) + 0.2 * (x > 0.4)
        return W.conserved_1d(rho, 0.3 * np.cos(2 * np.pi * nx / 20 * x),
                              0.7 + 0.1 * np.sin(2 * np.pi * x))
    return spec, W.project_1d(spec, u0)


def _waves_2d(n):
    spec = W.Spec(dim=2, flux=W.EULER, nx=n, ny=n, t_end=10.0)

    def u0(x, y, i, j):
        s = 0.7 + 0.2 * np.sin(10 * np.pi * (x + y) + 0.4) + 0.1 * (x > 0.4)
        u, v = 0.3 * np.cos(8 * np.pi * x), -0.2 * np.sin(6 * np.pi * y)
        p = 0.8 + 0.1 * np.cos(8 * np.pi * (x - y))
        return np.stack([s, s * u, s * v, p / 0.4 + 0.5 * s * (u * u + v * v)])
    return spec, W.project_2d(spec, u0)


def _config(dim, weights, own, **kw):
    cfg = hw.default_config(dim, weights=weights, **kw)
    if own:
        for m, g in enumerate(GAMMA[dim]):
            cfg.gamma_lin[m] = g
    return cfg


def _check(spec, st, cfg):
    with hw.Handle([spec], cfg) as h:
        h.set_state(0, st)
        ax, ay = h.alpha(0)
        L, Uh = h.rhs(0)
        dt = h.step(want_dt=True)[0]
        got, _ = h.get_state(0)
    p = oproblem(spec, cfg)
    ay = ay if spec.dim == 2 else 0.0
    S, SL = natural_scales(spec, st), rhs_scales(spec, st, ax, ay)
    # one evaluation or step: 1e-12 in FP64 and 2e-5 in single precision (some
    # hundred roundings of 6e-8 next to a jump), or ten times what the oracle
    # itself moves when its input is perturbed at the path's rounding level
    rel, floor = (1e-15, 1e-12) if cfg.precision == hw.F64 else (1e-7, 2e-5)
    for out, sc, fn in [(Uh, S, lambda s: O.rhs(p, s, ax, ay)[1]),
                        (L, SL, lambda s: O.rhs(p, s, ax, ay)[0]),
                        (got, S, lambda s: O.step(p, s, ax, ay, dt))]:
        sens = oracle_sensitivity(fn, st, sc, rel=rel)
        ok, err, bar = within_conditioning(out, fn(st), sc, sens, floor)
        assert ok, (err, bar)
    # the form matters on these data: the default's operator is far away
    q = oproblem(spec, hw.default_config(spec.dim, precision=cfg.precision, gauss_q=cfg.gauss_q,
                                         characteristic=cfg.characteristic,
                                         alpha_stage=cfg.alpha_stage))
    other, mine = O.rhs(q, st, ax, ay)[0], O.rhs(p, st, ax, ay)[0]
    same = cfg.weights == hw.W_PAPER and spec.dim == 1   # prints the default's form
    assert same or scaled_err(other, mine, SL) > 1e-3


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64, hw.F32_KAHAN, hw.F32])
@pytest.mark.parametrize("charwise", [0, 1])
@pytest.mark.parametrize("nx,alpha_stage", [(200, 0), (600, 0), (300, 1)])
@pytest.mark.parametrize("name,weights,own", FORMS)
def test_weight_forms_1d(name, weights, own, nx, alpha_stage, charwise, prec):
    spec, st = _waves_1d(nx)
    _check(spec, st, _config(1, weights, own, precision=prec, characteristic=charwise,
                             alpha_stage=alpha_stage))


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64, hw.F32_KAHAN, hw.F32])
@pytest.mark.parametrize("q", [2, 3])
@pytest.mark.parametrize("charwise", [0, 1])
@pytest.mark.parametrize("name,weights,own", FORMS)
def test_weight_forms_2d(name, weights, own, charwise, q, prec):
    spec, st = _waves_2d(70)
    _check(spec, st, _config(2, weights, own, precision=prec, gauss_q=q, characteristic=charwise))


@pytest.mark.parametrize("prec", [hw.F64, hw.F32_ACC64])
@pytest.mark.parametrize("name,weights,own", FORMS)
def test_weight_forms_of_a_scalar_law(name, weights, own, prec):
    spec, st = W.burgers_2d(65)
    st = st + 0.4 * (np.arange(65) > 30)[None, None, None, :] * (np.arange(3) == 0)[:, None, None, None]
    _check(spec, st, _config(2, weights, own, precision=prec, gauss_q=3))
