"""The oracle in 80-bit arithmetic (x87 long double), for what FP64 rounds too
coarsely to show: its C source with every `double` widened, every decimal
constant made long double and the mathematical functions of that type, behind
the same calls on double arrays."""
import ctypes as C
import os
import re
import subprocess
import tempfile

import numpy as np

import oracle as O

_SHIM = """
typedef struct {
    int dim, flux, nx, ny;
    double xlo, xhi, ylo, yhi;
    int bc_x, bc_y;
    double gas_gamma, adv[2];
    int gauss_q, weights;
    double gamma_lin[5], eps;
    int charwise, smoothness, alpha_stage;
} narrow_problem;

int ext_rhs(const narrow_problem* d, const double* state, double ax, double ay, double* L_out,
            double* Uhat_out, long n) {
    orc_problem p = {.dim = d->dim, .flux = d->flux, .nx = d->nx, .ny = d->ny, .xlo = d->xlo,
                     .xhi = d->xhi, .ylo = d->ylo, .yhi = d->yhi, .bc_x = d->bc_x, .bc_y = d->bc_y,
                     .gas_gamma = d->gas_gamma, .adv = {d->adv[0], d->adv[1]},
                     .gauss_q = d->gauss_q, .weights = d->weights, .eps = d->eps,
                     .charwise = d->charwise, .smoothness = d->smoothness,
                     .alpha_stage = d->alpha_stage};
    for (int m = 0; m < 5; ++m) p.gamma_lin[m] = d->gamma_lin[m];
    long double* w = malloc(3 * n * sizeof *w);
    if (!w) return -1;
    for (long i = 0; i < n; ++i) w[i] = state[i];
    const int rc = orc_rhs(&p, w, ax, ay, w + n, w + 2 * n);
    for (long i = 0; i < n; ++i) {
        L_out[i] = (double)w[n + i];
        Uhat_out[i] = (double)w[2 * n + i];
    }
    free(w);
    return rc;
}
"""
_lib = None


def _widen(text):
    text = re.sub(r"(?<![\w.])(\d+\.\d*(?:[eE][-+]?\d+)?)(?![\w.])", r"\1L", text)
    text = re.sub(r"\bdouble\b", "long double", text)
    return re.sub(r"\b(sqrt|fabs|pow)\(", r"\1l(", text)


def _load():
    global _lib
    if _lib is None:
        here = os.path.dirname(O.SRC_PATH)
        with tempfile.TemporaryDirectory() as d:
            with open(os.path.join(here, "hweno_oracle.h")) as f, \
                    open(os.path.join(d, "hweno_oracle.h"), "w") as g:
                g.write(_widen(f.read()))
            with open(O.SRC_PATH) as f, open(os.path.join(d, "extended.c"), "w") as g:
                g.write(_widen(f.read()) + _SHIM)
            so = os.path.join(d, "extended.so")
            subprocess.run(["gcc", "-O2", "-std=c99", "-ffp-contract=off", "-fopenmp", "-shared",
                            "-fPIC", "-o", so, os.path.join(d, "extended.c"), "-lm"], check=True)
            _lib = C.CDLL(so)
    return _lib


def rhs(p, state, ax, ay):
    """L and U-hat of a state, as the oracle's rhs."""
    state = np.ascontiguousarray(state, dtype=np.float64)
    L, Uh = np.empty_like(state), np.empty_like(state)
    D, c = C.POINTER(C.c_double), p._c()
    rc = _load().ext_rhs(C.byref(c), state.ctypes.data_as(D), C.c_double(ax), C.c_double(ay),
                         L.ctypes.data_as(D), Uh.ctypes.data_as(D), C.c_long(state.size))
    assert rc == 0, rc
    return L, Uh
